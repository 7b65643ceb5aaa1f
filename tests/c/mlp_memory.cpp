// The gradient of a deep network on a device whose memory does not hold a delta per layer:
// the library's allocations are answered here and refused above a limit.
#include <dlfcn.h>
#include <hip/hip_runtime_api.h>

#include <cmath>
#include <cstdio>
#include <vector>

#include "riccsd.h"

static size_t g_limit = ~size_t{0};
static int g_refused = 0;
extern "C" hipError_t hipMallocAsync(void** p, size_t bytes, hipStream_t s) {
  static auto real = reinterpret_cast<hipError_t (*)(void**, size_t, hipStream_t)>(dlsym(RTLD_NEXT, "hipMallocAsync"));
  if (bytes > g_limit) return ++g_refused, hipErrorOutOfMemory;
  return real(p, bytes, s);
}

int main() {
  const int d = 8, h = 256, layers = 6;
  const long n = 4096;
  std::vector<float> x(n * d), y(n);
  unsigned u = 1;
  auto next = [&] { return static_cast<float>((u = u * 1664525u + 1013904223u) >> 8) / 8388608.f - 1.f; };
  for (float& v : x) v = next();
  for (float& v : y) v = next();
  float *X, *Y;
  if (hipMalloc(reinterpret_cast<void**>(&X), x.size() * 4) != hipSuccess ||
      hipMalloc(reinterpret_cast<void**>(&Y), y.size() * 4) != hipSuccess)
    return 2;
  (void)hipMemcpy(X, x.data(), x.size() * 4, hipMemcpyHostToDevice);
  (void)hipMemcpy(Y, y.data(), y.size() * 4, hipMemcpyHostToDevice);
  std::vector<float> g[2];
  float loss[2];
  for (int k = 0; k < 2; ++k) {
    // activations and two deltas take 34 MB, a delta per layer 17 MB more, the rest 8 MB
    g_limit = k == 0 ? ~size_t{0} : size_t{45} << 20;
    ri_mlp* net = ri_mlp_create(d, h, layers);
    const size_t np = ri_mlp_num_params(net);
    float* G;
    if (hipMalloc(reinterpret_cast<void**>(&G), np * 4) != hipSuccess) return 2;
    if (ri_mlp_init(net, 7, nullptr) != RI_OK) return 2;
    const int rc = ri_mlp_gradient(net, X, Y, n, G, &loss[k], nullptr);
    if (rc != RI_OK) {
      std::printf("gradient %d: status %d (%s)\n", k, rc, ri_last_error_msg());
      return 1;
    }
    g[k].resize(np);
    (void)hipMemcpy(g[k].data(), G, np * 4, hipMemcpyDeviceToHost);
    ri_mlp_destroy(net);
  }
  float big = 0.f, diff = 0.f;
  for (size_t i = 0; i < g[0].size(); ++i) {
    big = std::fmax(big, std::fabs(g[0][i]));
    diff = std::fmax(diff, std::fabs(g[0][i] - g[1][i]));
  }
  std::printf("refused %d, largest gradient %g, difference %g, loss %g %g\n", g_refused, big, diff, loss[0], loss[1]);
  // both sum 4096 FP32 terms in their own order: within 1e-4 of the largest value
  if (g_refused != 1 || !(diff <= 1e-4f * big) || !(std::fabs(loss[0] - loss[1]) <= 1e-4f * loss[0])) return 1;
  std::printf("mlp memory ok\n");
  return 0;
}
