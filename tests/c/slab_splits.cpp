// Host check of the ladder's partial-sum buffers (no GPU): built with SOURCE set to one of
// the library's ladder sources, whose own plan and split rule it walks slab by slab as the
// ladder and its exchange-symmetric form do.  The device queries are answered here, so that
// the rule sees every occupancy the contraction kernels can have.
#include <cstdio>

#include SOURCE

static int g_wgs = 2;  // resident workgroups per CU
extern "C" hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
extern "C" hipError_t hipDeviceGetAttribute(int* x, hipDeviceAttribute_t, int) { return *x = 256, hipSuccess; }
extern "C" hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
  return *n = g_wgs, hipSuccess;
}

using namespace ri::ppl;
static long fails = 0, slabs = 0, capped = 0;

// One slab: `rows` rows summed over K slots.  rule: the split count the rule asks for
// without a buffer, and its slots per split.
template <class P, class Rule>
static void slab(const P& p, bool minus, long rows, long K, bool must_equal, Rule rule, int o, int v) {
  long kz = 0, kz0 = 0;
  const long held = minus ? p.zrows_m : p.zrows_p;
  const long z = slab_splits(p, minus, rows, K, kz), z0 = rule(minus, rows, K, kz0);
  ++slabs;
  if (z0 * rows > held) ++capped;
  const bool ok = z >= 1 && z * rows <= held && kz > 0 && z * kz >= K && (z - 1) * kz < K &&
                  ((z0 * rows > held && !must_equal) || (z == z0 && kz == kz0));
  if (ok) return;
  if (++fails <= 10)
    std::printf("o=%d v=%d %c: %ld rows over %ld slots: %ld splits of %ld (rule: %ld of %ld), %ld rows held\n", o, v,
                minus ? '-' : '+', rows, K, z, kz, z0, kz0, held);
}
// The slabs of plan p: all slots summed (the plain ladder, where the rule's own count always
// fits and is kept) or those from the slab's first on (the exchange-symmetric form).
template <class P, class Rule>
static void walk(const P& p, bool sym, Rule rule, int o, int v) {
  for (long s0 = 0; s0 < p.nbp; s0 += p.slab_bp) {
    const long rows = std::min(p.nbp - s0, p.slab_bp) * 256, K = sym ? p.K - s0 * 256 : p.K;
    slab(p, false, rows, K, !sym, rule, o, v);
    if (p.pm > 0) slab(p, true, rows, K, !sym, rule, o, v);
  }
}

static void check(int o, int v, long sym_slab_bp) {
#ifdef SPLIT_BF16
  MPlan p;
  if (!make_mplan(o, v, 3 * v, p)) return;
  auto rule = [&](bool m, long rows, long K, long& kz) {
    return contract_splits(m ? p.wide_m : p.wide_p, m ? p.ntw_m : p.ntw_p, m ? p.NM : p.NP, rows, K, 0, kz);
  };
  walk(p, false, rule, o, v);
  p.slab_bp = std::max(1L, std::min(sym_slab_bp, p.nbp));
  size_mplan(p);
  walk(p, true, rule, o, v);
#else
  for (size_t es : {size_t(8), size_t(4)}) {
    Plan p;
    auto rule = [&](bool m, long rows, long K, long& kz) {
      return contract_splits(m ? p.NM : p.NP, m ? p.ntw_m : p.ntw_p, rows, K, p.esize, p.fixed, 0, kz);
    };
    if (!make_plan(o, v, 3 * v, es, p)) return;
    walk(p, false, rule, o, v);
    make_plan(o, v, 3 * v, es, p, true);
    p.slab_bp = sym_slab_bp;
    size_plan(p, true);
    walk(p, true, rule, o, v);
  }
#endif
}

int main() {
  for (g_wgs = 1; g_wgs <= 4; ++g_wgs)
    for (int v = 16; v <= 320; v += v % 16 == 0 ? 1 : 15)  // every padded size, from both ends
      for (int o = 1; o <= v / 5; ++o) {
        const long nb = (v + TB - 1) / TB, nbp = nb * (nb + 1) / 2;
        check(o, v, (nbp + 7) / 8);  // the default of eight slabs
        if (o % 3 == 0) check(o, v, (nbp + 2) / 3);
      }
  std::printf("%ld slabs, %ld with fewer splits than asked for\n", slabs, capped);
  if (capped == 0) ++fails;  // the sweep holds such slabs
  if (fails == 0) std::printf("slab splits ok\n");
  return fails == 0 ? 0 : 1;
}
