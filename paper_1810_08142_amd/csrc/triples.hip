// Perturbative triples energy E_(T) of closed-shell CCSD(T) (Sec. II.A): FP64, with an
// FP32 option for the term GEMMs.
//
//   E_(T) = sum_{ijk} sum_{abc} (4 W^{abc}_{ijk} + W^{bca}_{ijk} + W^{cab}_{ijk})
//                               (V^{abc}_{ijk} - V^{cba}_{ijk}) / (3 D^{abc}_{ijk}),
//   W^{abc}_{ijk} = P^{abc}_{ijk} X(ijk, abc),
//   X(ijk, abc)   = sum_d (bd|ai) t^{cd}_{kj} - sum_l (ck|jl) t^{ab}_{il},
//   V^{abc}_{ijk} = W^{abc}_{ijk} + (jb|kc) t^a_i + (ia|kc) t^b_j + (ia|jb) t^c_k,
//   D^{abc}_{ijk} = e_i + e_j + e_k - e_a - e_b - e_c,
//
// (v^{pq}_{rs} = (pr|qs); P sums the six simultaneous permutations of the column pairs
// (i, a), (j, b), (k, c)).  W and V are invariant under those simultaneous
// permutations, so one triplet i <= j <= k gives W and V for every ordering of it:
// W_{i'j'k'} is W_{ijk} with its virtual indices permuted the same way.  The summand
// itself is not invariant (W^{bca}, W^{cab} and V^{cba} relabel the virtuals alone),
// so the energy kernel evaluates it for each distinct ordering (i', j', k') from the
// one W and V, reading them through permuted tiles.
//
// Triplets are taken in batches.  The six terms of P come in pairs with one third virtual
// z: X(p, q, r; x, y, z) and X(q, p, r; y, x, z), both [x][y][z] with a summed index of their
// own, so each pair is one GEMM over the two summed indices one after the other (the second
// A read with its rows (x, y) exchanged).  Per batch: one launch of three such GEMMs per
// triplet on the library's MFMA engine (FP64; with FP32 terms two GEMMs per pair, one after
// the other, the second adding to the first), each writing its pair's sum in its
// own natural layout (contiguous output rows; the o-sized sum of a term rides along as extra
// columns of the summed index), and one tiled kernel that symmetrises the three into W,
// forms V = W + the t1 terms and sums the energy in a fixed order, all in LDS.  The GEMM
// operands (with (yd|xp) and (zr|ql) from the RI factors) and (ia|jb) are built once.
#include <cmath>
#include <vector>

#include "gemm.h"

namespace ri {
namespace trip {

constexpr int TE = 8;  // tile edge of the energy kernel

// element m of permutation p of (0, 1, 2): p in the order 012 021 102 120 201 210, the
// 18 two-bit elements packed in that order
__host__ __device__ constexpr int perm_at(int p, int m) {
  return static_cast<int>((0x192261624ull >> (2 * (3 * p + m))) & 3ull);
}
// index of the permutation (e0, e1, e2) in the order of perm_at
__host__ __device__ constexpr int perm_index(int e0, int e1) { return 2 * e0 + (e1 > e0 ? e1 - 1 : e1); }
// p o q: element m is element q(m) of p
__host__ __device__ constexpr int perm_mul(int p, int q) {
  return perm_index(perm_at(p, perm_at(q, 0)), perm_at(p, perm_at(q, 1)));
}
__host__ __device__ constexpr int perm_inv(int p) {
  return perm_index(perm_at(p, 0) == 0 ? 0 : perm_at(p, 1) == 0 ? 1 : 2,
                    perm_at(p, 0) == 1 ? 0 : perm_at(p, 1) == 1 ? 1 : 2);
}

// Energy of the triplets of a batch, W and V formed on the way.
//
//   W[a][b][c] = sum over p in {012, 021, 120} of Y_p[y0][y1][y2], y_m = (a, b, c)[perm(p, m)]
//   (the three pair sums of P, each computed in its own natural layout),
//   V = W + (jb|kc) t^a_i + (ia|kc) t^b_j + (ia|jb) t^c_k.
//
// One block per unordered triple of 8-wide tiles {A, B, C} (A <= B <= C, packed in tiles[]
// as A | B << 10 | C << 20) and triplet.  It reads the 8^3 tiles of the three Y at the six
// orientations (every element of Y once over the launch, 18 loads per thread issued
// together), sums them through LDS (all global accesses run along the last index) and
// keeps the six orientations of W and V there: orientation p holds W[Z_p0 + u][Z_p1 + w]
// [Z_p2 + z] for Z = (A, B, C) in elements.  Then it evaluates every distinct ordering of
// the tile triple: at (a, b, c) the six permuted elements of W and of V are read once and
// serve all orderings (i', j', k') of the triplet, ordering x taking W'^{abc} from
// permutation x^-1 and W'^{bca}, W'^{cab}, V'^{cba} from it followed by the relabelling.
// LDS tiles have strides 73, 9, 1 (at most two lanes of a permuted read share a bank).
// Bound by the read of Y (24 v^3 bytes a triplet); at o=12 v=120 a triplet takes 19.5 us
// (assembling six terms and summing in two kernels with W and V in memory: 94 us).
// part[blockIdx.y * gridDim.x + blockIdx.x].  grid (tile triples, triplets), block 512.
constexpr int LS0 = 73, LS1 = 9, LT = 584;
// the permutations whose natural layouts hold the pairs: 012, 021, 120
__host__ __device__ constexpr int term(int p) { return p == 2 ? 3 : p; }
struct Trip {
  int i, j, k;
};
// Summand of one (a, b, c) over the distinct orderings of a triplet (i' = x(0)-th of i, j, k
// and so on), from the permuted elements of W and V.  KIND: 1 for i == j, plus 2 for j == k;
// of the permutations that give one ordering the first is taken.
template <int KIND>
__device__ inline double orderings(const double (&wv)[6], const double (&vv)[6]) {
  double sum = 0.0;
#pragma unroll
  for (int x = 0; x < 6; ++x) {
    if (KIND == 3 ? x > 0 : KIND == 1 ? perm_mul(2, x) < x : KIND == 2 ? perm_mul(1, x) < x : false) continue;
    const int inv = perm_inv(x);
    sum += (4.0 * wv[inv] + wv[perm_mul(3, inv)] + wv[perm_mul(4, inv)]) * (vv[inv] - vv[perm_mul(5, inv)]);
  }
  return sum;
}
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4))) void energy_tiles(
    const double* __restrict__ Y, const double* __restrict__ K, const double* __restrict__ t1,
    const double* __restrict__ eps, int o, int v, const Trip* __restrict__ trips, const int* __restrict__ tiles,
    double* __restrict__ part) {
  __shared__ double st[3 * LT];
  __shared__ double tw[6 * LT];
  __shared__ double tv[6 * LT];
  const int code = tiles[blockIdx.x];
  const int bt[3] = {code & 1023, (code >> 10) & 1023, (code >> 20) & 1023};
  const Trip tr = trips[blockIdx.y];
  const long v3 = static_cast<long>(v) * v * v;
  Y += 3 * v3 * blockIdx.y;
  const int t = threadIdx.x, u = t >> 6, w = (t >> 3) & 7, z = t & 7;
  const int x[3] = {u, w, z};
  // element of a Y tile: coordinate m of the thread in the block of virtuals bt[q]; past the
  // edge the last element is read (never used)
  int e[3][3];
#pragma unroll
  for (int q = 0; q < 3; ++q)
#pragma unroll
    for (int m = 0; m < 3; ++m) e[q][m] = min(bt[q] * TE + x[m], v - 1);
  int L[6];  // position of the thread's permuted coordinates in an LDS tile
#pragma unroll
  for (int p = 0; p < 6; ++p) L[p] = x[perm_at(p, 0)] * LS0 + x[perm_at(p, 1)] * LS1 + x[perm_at(p, 2)];
  double y[6][3];  // [orientation][pair]
#pragma unroll
  for (int sg = 0; sg < 6; ++sg)
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      const int q = perm_mul(sg, term(p));
      y[sg][p] = Y[p * v3 + (static_cast<long>(e[perm_at(q, 0)][0]) * v + e[perm_at(q, 1)][1]) * v + e[perm_at(q, 2)][2]];
    }
  auto Kx = [&](int i1, int p1, int i2, int p2) { return K[((static_cast<long>(i1) * v + p1) * o + i2) * v + p2]; };
#pragma unroll
  for (int sg = 0; sg < 6; ++sg) {
    double acc = 0.0;
    __syncthreads();
#pragma unroll
    for (int p = 0; p < 3; ++p) st[p * LT + L[0]] = y[sg][p];
    __syncthreads();
#pragma unroll
    for (int p = 0; p < 3; ++p) acc += st[p * LT + L[term(p)]];
    const int a = e[perm_at(sg, 0)][0], b = e[perm_at(sg, 1)][1], c = e[perm_at(sg, 2)][2];
    tw[sg * LT + L[0]] = acc;
    tv[sg * LT + L[0]] = acc + Kx(tr.j, b, tr.k, c) * t1[tr.i * v + a] + Kx(tr.i, a, tr.k, c) * t1[tr.j * v + b] +
                         Kx(tr.i, a, tr.j, b) * t1[tr.k * v + c];
  }
  __syncthreads();
  const int kind = (tr.i == tr.j ? 1 : 0) + (tr.j == tr.k ? 2 : 0);
  const double eo = eps[tr.i] + eps[tr.j] + eps[tr.k];
  double acc = 0.0;
#pragma unroll
  for (int sg = 0; sg < 6; ++sg) {
    // skip an ordering of the tile triple that repeats an earlier one (equal tiles)
    const int k0 = bt[perm_at(sg, 0)], k1 = bt[perm_at(sg, 1)], k2 = bt[perm_at(sg, 2)];
    bool dup = false;
#pragma unroll
    for (int s2 = 0; s2 < sg; ++s2)
      dup = dup || (bt[perm_at(s2, 0)] == k0 && bt[perm_at(s2, 1)] == k1 && bt[perm_at(s2, 2)] == k2);
    if (dup) continue;
    const int a = k0 * TE + u, b = k1 * TE + w, c = k2 * TE + z;
    if (a >= v || b >= v || c >= v) continue;
    // element (a, b, c) of orientation sg; read through permutation p it comes from tile
    // sg o p at the thread's coordinates permuted by p
    double wv[6], vv[6];
#pragma unroll
    for (int p = 0; p < 6; ++p) {
      wv[p] = tw[perm_mul(sg, p) * LT + L[p]];
      vv[p] = tv[perm_mul(sg, p) * LT + L[p]];
    }
    const double d = eo - (eps[o + a] + eps[o + b] + eps[o + c]);
    const double sum = kind == 0 ? orderings<0>(wv, vv) : kind == 1 ? orderings<1>(wv, vv)
                     : kind == 2 ? orderings<2>(wv, vv) : orderings<3>(wv, vv);
    acc += sum / (3.0 * d);
  }
  __syncthreads();  // the reduction reuses the staging tiles
  st[t] = acc;
  __syncthreads();
  for (int s = 256; s > 0; s >>= 1) {
    if (t < s) st[t] += st[t + s];
    __syncthreads();
  }
  if (t == 0) part[static_cast<long>(blockIdx.y) * gridDim.x + blockIdx.x] = st[0];
}

// out[b] = sum of part[b n .. b n + n) in a fixed order, b = blockIdx.x
__global__ __launch_bounds__(256) void sum_parts(const double* __restrict__ part, long n, double* out) {
  __shared__ double red[256];
  part += blockIdx.x * n;
  double acc = 0.0;
  for (long x = threadIdx.x; x < n; x += 256) acc += part[x];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[blockIdx.x] = red[0];
}

}  // namespace trip
}  // namespace ri

using namespace ri;

extern "C" {

double ri_ccsd_triples_flops(int o, int v) {
  if (o <= 0 || v <= 0) return 0.0;
  const double trip = o * (o + 1.0) * (o + 2.0) / 6.0, v3 = static_cast<double>(v) * v * v;
  return trip * 6.0 * 2.0 * v3 * (v + o);
}

int ri_ccsd_triples_ex(const ri_system* sys, const double* t1, const double* t2, int precision, double* e_t,
                       void* stream) {
  clear_error();
  RI_TRY(cc::check_system(sys, "ri_ccsd_triples"));
  if (!t1 || !t2 || !e_t) {
    set_error("ri_ccsd_triples: null pointer argument");
    return RI_E_ARG;
  }
  if (precision != RI_PREC_FP64 && precision != RI_PREC_FP32) {
    set_error("ri_ccsd_triples: precision %d is not FP64 or FP32", precision);
    return RI_E_ARG;
  }
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int o = sys->o, v = sys->v, Q = sys->naux, n = o + v;
  const int vo = (v + o + 15) / 16 * 16;  // summed index of a term, padded with zeros to 16
  const long nn = static_cast<long>(n) * n, vv = static_cast<long>(v) * v, v3 = vv * v;
  const int nt = (v + trip::TE - 1) / trip::TE;
  if (nt > 1023) {
    set_error("ri_ccsd_triples: v = %d is too large for the energy tiles", v);
    return RI_E_ARG;
  }
  const long ntri = static_cast<long>(nt) * (nt + 1) * (nt + 2) / 6;  // energy tile triples
  const long ntrip = static_cast<long>(o) * (o + 1) * (o + 2) / 6;
  // Each term of P, X(p, q, r; x, y, z) = sum_d (yd|xp) t2[r][q][z][d] - sum_l (zr|ql) t2[p][l][x][y],
  // is one GEMM over the combined index e = (d, then l):
  //   A[p][x][y][e] = (yd|xp) for e = d < v,  t2[p][l][x][y] for e = v + l,
  //   Bt[r][q][z][e] = t2[r][q][z][d] for e = d < v,  -(zr|ql) for e = v + l.
  // Buffers: A [o][v][v][v+o], Bt [o][o][v][v+o], J [o][o][v][o], K [o][v][o][v],
  // Y [batch][3][v][v][v] (the pair sums), tile partials, triplet sums, the GEMMs' offsets,
  // the triplets, the tile triples.
  // Batch: GEMM tiles (128 x 128) for about four rounds of the chip's two workgroups per CU,
  // at most 16 triplets and 2 GiB of Y.  Of one to three triplets less than four rounds need,
  // and up to that, the count whose last round is fullest (v = 120, 339 tiles a triplet: six
  // triplets are 3.97 rounds, seven 4.63).
  const long tiles = 3 * ((vv + 127) / 128) * ((v + 127) / 128);
  const long most = std::max(1L, std::min({(2048 + tiles - 1) / tiles, 16L, (1L << 28) / (3 * v3), ntrip}));
  long nb = most;
  auto rounds = [&](long b) { return (b * tiles + 511) / 512; };
  for (long b = most - 1; b >= std::max(1L, most - 3); --b)
    if (rounds(b) * nb < rounds(nb) * b) nb = b;  // fewer rounds per triplet
  const size_t nA = static_cast<size_t>(o) * vv * vo, nBt = static_cast<size_t>(o) * o * v * vo,
               nJ = static_cast<size_t>(o) * o * v * o, nK = static_cast<size_t>(o) * v * o * v;
  auto even = [](size_t x) { return (x + 1) / 2 * 2; };
  const size_t bytes = (even(nA) + even(nBt) + even(nJ) + even(nK) + even(3 * nb * static_cast<size_t>(v3)) +
                        nb * ntri + ntrip + 15 * static_cast<size_t>(ntrip)) * sizeof(double) +
                       ntrip * sizeof(trip::Trip) + ntri * sizeof(int);
  void* buf = nullptr;
  RI_TRY(dev_alloc(&buf, bytes, s));
  double* A = static_cast<double*>(buf);
  double* Bt = A + even(nA);
  double* J = Bt + even(nBt);
  double* K = J + even(nJ);
  double* Y = K + even(nK);
  double* part = Y + even(3 * nb * static_cast<size_t>(v3));
  double* et = part + nb * ntri;
  long* items = reinterpret_cast<long*>(et + ntrip);
  trip::Trip* tp = reinterpret_cast<trip::Trip*>(items + 15 * ntrip);
  int* tl = reinterpret_cast<int*>(tp + ntrip);
  std::vector<int> tiles_host;
  tiles_host.reserve(ntri);
  for (int ta = 0; ta < nt; ++ta)
    for (int tb = ta; tb < nt; ++tb)
      for (int tc = tb; tc < nt; ++tc) tiles_host.push_back(ta | (tb << 10) | (tc << 20));
  // the triplets in order and, per triplet and pair, the offsets of its GEMM: (p, q, r) = the
  // triplet and (x, y, z) = (a, b, c), both permuted by the pair's m; Y_m [x][y][z]
  std::vector<trip::Trip> trips;
  std::vector<long> items_host;
  trips.reserve(ntrip);
  items_host.reserve(15 * ntrip);
  const long sA0 = vv * vo, sB1 = static_cast<long>(v) * vo;
  for (int i = 0; i < o; ++i)
    for (int j = i; j < o; ++j)
      for (int k = j; k < o; ++k) {
        const int x3[3] = {i, j, k};
        for (int h = 0; h < 3; ++h) {
          const int m = trip::term(h);
          const long pp = x3[trip::perm_at(m, 0)], qq = x3[trip::perm_at(m, 1)], rr = x3[trip::perm_at(m, 2)];
          const long at[5] = {pp * sA0, (rr * o + qq) * sB1, qq * sA0, (rr * o + pp) * sB1,
                              (static_cast<long>(trips.size()) % nb * 3 + h) * v3};
          items_host.insert(items_host.end(), at, at + 5);
        }
        trips.push_back(trip::Trip{i, j, k});
      }
  int rc = RI_OK;
  {
    GemmArena arena;
    arena.s = s;
    const double* B = sys->B;
    // B views (occupied first): vv, vo, oo, ov blocks of [Q][n][n]
    const Tensor Bvv(B + static_cast<long>(o) * n + o, {Q, v, v}, {nn, n, 1});
    const Tensor Bvo(B + static_cast<long>(o) * n, {Q, v, o}, {nn, n, 1});
    const Tensor Boo(B, {Q, o, o}, {nn, n, 1});
    const Tensor Bov(B + o, {Q, o, v}, {nn, n, 1});
    const long sA2 = vo, sA1 = static_cast<long>(v) * vo;                    // strides of A
    const long sB2 = vo, sB0 = static_cast<long>(o) * v * vo;  // of Bt
    do {
      if ((rc = check_hip(hipMemcpyAsync(tl, tiles_host.data(), ntri * sizeof(int), hipMemcpyHostToDevice, s),
                          "triples tiles")))
        break;
      if ((rc = check_hip(hipMemcpyAsync(tp, trips.data(), ntrip * sizeof(trip::Trip), hipMemcpyHostToDevice, s),
                          "triples list")))
        break;
      if ((rc = check_hip(hipMemcpyAsync(items, items_host.data(), 15 * ntrip * sizeof(long), hipMemcpyHostToDevice, s),
                          "triples offsets")))
        break;
      // zero padding of the summed index (columns v + o .. vo - 1)
      if ((rc = check_hip(hipMemsetAsync(A, 0, (even(nA) + even(nBt)) * sizeof(double), s), "triples clear"))) break;
      // A[p][x][y][d] = (yd|xp)
      if ((rc = einsum("Qyd,Qxp->pxyd", 1.0, Bvv, Bvo, 0.0, Tensor(A, {o, v, v, v}, {sA0, sA1, sA2, 1}), arena,
                       s)))
        break;
      // A[p][x][y][v + l] = t2[p][l][x][y]
      if ((rc = axpby_perm("plxy->pxyl", 1.0, Tensor(t2, {o, o, v, v}), 0.0,
                           Tensor(A + v, {o, v, v, o}, {sA0, sA1, sA2, 1}), s)))
        break;
      // J[r][q][z][l] = (zr|ql); Bt[r][q][z][d] = t2[r][q][z][d], Bt[r][q][z][v + l] = -J[r][q][z][l]
      if ((rc = einsum("Qzr,Qql->rqzl", 1.0, Bvo, Boo, 0.0, Tensor(J, {o, o, v, o}), arena, s))) break;
      if ((rc = axpby_perm("rqzd->rqzd", 1.0, Tensor(t2, {o, o, v, v}), 0.0,
                           Tensor(Bt, {o, o, v, v}, {sB0, sB1, sB2, 1}), s)))
        break;
      if ((rc = axpby_perm("rqzl->rqzl", -1.0, Tensor(J, {o, o, v, o}), 0.0,
                           Tensor(Bt + v, {o, o, v, o}, {sB0, sB1, sB2, 1}), s)))
        break;
      // K[i][a][j][b] = (ia|jb)
      if ((rc = einsum("Qia,Qjb->iajb", 1.0, Bov, Bov, 0.0, Tensor(K, {o, v, o, v}), arena, s))) break;
      // Y_m[x][y][z] = sum_e A[p][x][y][e] Bt[r][q][z][e] + A[q][y][x][e] Bt[r][p][z][e]
      gemm::GemmDesc g{};
      g.M = vv;
      g.N = v;
      g.K = vo;
      g.M2 = v;
      g.N2 = v;
      g.K2 = 1;
      g.K3 = vo;
      g.a = A;
      g.am1 = sA1;
      g.am2 = sA2;
      g.ak3 = 1;
      g.b = Bt;
      g.bn2 = vo;
      g.bk3 = 1;
      g.c = Y;
      g.cm1 = vv;
      g.cm2 = v;
      g.cn2 = 1;
      g.alpha = 1.0;
      g.beta = 0.0;
      for (long t0 = 0; t0 < ntrip && rc == RI_OK; t0 += nb) {
        const long n_t = std::min(nb, ntrip - t0);
        if (precision == RI_PREC_FP64) {
          ProfScope ps(s, "xye,ze->xyz", 12.0 * n_t * static_cast<double>(v3) * vo);
          rc = gemm::run_pairs(g, v + o, static_cast<int>(3 * n_t), items + 15 * t0, s);
        } else {
          for (long x = 0; x < 3 * n_t && rc == RI_OK; ++x) {
            const long* at = &items_host[15 * t0 + 5 * x];
            const Tensor Yt(Y + at[4], {v, v, v});
            rc = einsum("xye,ze->xyz", 1.0, Tensor(A + at[0], {v, v, vo}, {sA1, sA2, 1}),
                        Tensor(Bt + at[1], {v, vo}, {sB2, 1}), 0.0, Yt, arena, s, precision);
            if (rc) break;
            rc = einsum("xye,ze->xyz", 1.0, Tensor(A + at[2], {v, v, vo}, {sA2, sA1, 1}),
                        Tensor(Bt + at[3], {v, vo}, {sB2, 1}), 1.0, Yt, arena, s, precision);
          }
        }
        if (rc) break;
        ProfScope ps(s, "triples_energy", 0.0, 24.0 * n_t * v3);
        trip::energy_tiles<<<dim3(static_cast<unsigned>(ntri), static_cast<unsigned>(n_t)), 512, 0, s>>>(
            Y, K, t1, sys->eps, o, v, tp + t0, tl, part);
        trip::sum_parts<<<static_cast<unsigned>(n_t), 256, 0, s>>>(part, ntri, et + t0);
        rc = check_launch("triples_energy");
      }
      if (rc) break;
      std::vector<double> h(ntrip);
      if ((rc = check_hip(hipMemcpyAsync(h.data(), et, ntrip * sizeof(double), hipMemcpyDeviceToHost, s),
                          "triples copy")))
        break;
      if ((rc = check_hip(hipStreamSynchronize(s), "triples sync"))) break;
      double e = 0.0;
      for (double x : h) e += x;
      if (!std::isfinite(e)) {
        set_error("ri_ccsd_triples: energy is not finite");
        rc = RI_E_NUMERIC;
        break;
      }
      *e_t = e;
    } while (false);
  }
  dev_free(buf, s);
  return rc;
}

int ri_ccsd_triples(const ri_system* sys, const double* t1, const double* t2, double* e_t, void* stream) {
  return ri_ccsd_triples_ex(sys, t1, t2, RI_PREC_FP64, e_t, stream);
}

}  // extern "C"
