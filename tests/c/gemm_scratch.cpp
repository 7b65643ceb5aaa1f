// Host check of the contractions' split-k scratch (no GPU): SOURCE is the library's own
// contraction source.
#include <cstdio>

#include SOURCE

using namespace ri::gemm;

// C [M][N] = A [M][K] B [K][N], row-major, the summed index in one level of extent K3 at least
static GemmDesc product(long M, long N, long K, long K3) {
  GemmDesc g{};
  g.M = M;
  g.N = N;
  g.K = K;
  g.M2 = M;
  g.N2 = N;
  g.K2 = K / K3;
  g.K3 = K3;
  g.am2 = K;
  g.ak2 = K3;
  g.ak3 = 1;
  g.bk2 = K3 * N;
  g.bk3 = N;
  g.bn2 = 1;
  g.cm2 = N;
  g.cn2 = 1;
  g.alpha = 1.0;
  return g;
}

int main() {
  int fails = 0;
  auto expect = [&](const char* what, const GemmDesc& g, int batch, bool some) {
    const size_t n = scratch_doubles(g, batch);
    if ((n > 0) == some) return;
    ++fails;
    std::printf("%s: %zu doubles of scratch\n", what, n);
  };
  // whole large tiles, from 256 of them on
  expect("2048 x 2048 x 2048", product(2048, 2048, 2048, 2048), 1, false);
  expect("2048 x 2176 x 65536", product(2048, 2176, 65536, 64), 1, false);
  expect("batch of four 1024 x 1024 x 4096", product(1024, 1024, 4096, 4096), 4, false);
  // fewer, split over the summed index
  expect("1920 x 1920 x 2048", product(1920, 1920, 2048, 2048), 1, true);
  expect("1024 x 1024 x 262144", product(1024, 1024, 262144, 512), 1, true);
  // the tiles of 64 x 64 fill the chip whole
  expect("2048 x 2048 x 2040", product(2048, 2048, 2040, 2040), 1, false);
  if (fails == 0) std::printf("gemm scratch ok\n");
  return fails;
}
