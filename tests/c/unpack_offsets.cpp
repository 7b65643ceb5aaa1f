// Host check of the unpack's element offsets (no GPU) against 64-bit ones, at column counts
// up to the largest that the ladder accepts, in the address an element is read from.
#include <cstdio>

#include "../../paper_1810_08142_amd/csrc/ppl_shared.h"

using namespace ri::ppl;

template <class T>
static long check(int ncol) {
  long fails = 0;
  const T* base = reinterpret_cast<const T*>(uintptr_t{1} << 40);
  for (int row = 0; row < 256; ++row)
    for (int col : {0, ncol / 2, ncol - 1}) {
      const auto got = reinterpret_cast<uintptr_t>(base + unpack_at(row, ncol, col));
      const auto want = (uintptr_t{1} << 40) + (static_cast<uintptr_t>(row) * ncol + col) * sizeof(T);
      if (got != want && ++fails <= 5)
        std::printf("%d columns of %zu bytes: row %d column %d\n", ncol, sizeof(T), row, col);
    }
  return fails;
}

int main() {
  long fails = 0;
  for (int o : {1, 2, 7, 16, 48, 300, 1000, 1447, 2047, 2048, 2051, 2052, 2100, 2900, 3500, 4095, 4096})
    for (int maxw : {9, 10, 16}) {
      int ntw, ncol;
      pick_ntw(o * (o + 1) / 2, maxw, 128, ntw, ncol);
      fails += check<float>(ncol) + check<double>(ncol);
    }
  if (fails == 0) std::printf("unpack offsets ok\n");
  return fails == 0 ? 0 : 1;
}
