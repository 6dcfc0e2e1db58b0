// short_memory.cpp -- a call whose neighbour rows cannot be allocated scans
// instead.  hipMalloc is taken over here: above a size it reports that memory is
// out.  Prints "ok" when the results are those of the unhindered call.
#include <dlfcn.h>
#include <hip/hip_runtime_api.h>

#include <cmath>
#include <cstdio>
#include <cstring>
#include <vector>

#include "ccm.h"

static size_t g_largest = ~(size_t)0;   // larger allocations fail
static int g_failed = 0;

extern "C" hipError_t hipMalloc(void** p, size_t n) {
  static const auto real = reinterpret_cast<hipError_t (*)(void**, size_t)>(
      dlsym(RTLD_NEXT, "hipMalloc"));
  if (n > g_largest) {
    ++g_failed;
    return hipErrorOutOfMemory;
  }
  return real(p, n);
}

static std::vector<double> call(ccm_ctx* c, const std::vector<double>& x,
                                const std::vector<double>& y, int r, ccm_status* st) {
  const int64_t L[2] = {1000, 3000};
  std::vector<double> rho(2 * 2 * (size_t)r, -7.0);
  *st = ccm(c, x.data(), y.data(), (int64_t)x.size(), 2, 1, L, 2, r, 5, nullptr, rho.data(),
            rho.data() + 2 * r, nullptr);
  return rho;
}

int main() {
  const int N = 4000;
  std::vector<double> x(N), y(N);
  x[0] = 0.4;
  y[0] = 0.2;
  for (int t = 0; t + 1 < N; ++t) {
    x[t + 1] = x[t] * (3.8 - 3.8 * x[t] - 0.02 * y[t]);
    y[t + 1] = y[t] * (3.5 - 3.5 * y[t] - 0.1 * x[t]);
  }
  ccm_ctx* c = nullptr;
  if (ccm_create(0, &c) != CCM_OK) return 2;
  ccm_status s0, s1, s2;
  const auto want = call(c, x, y, 100, &s0);   // the walks: over 12 MB at once
  (void)call(c, x, y, 1, &s1);                 // another plan, so that the next one is made anew
  g_largest = 10u << 20;
  const auto got = call(c, x, y, 100, &s2);
  const int failed = g_failed;
  g_largest = ~(size_t)0;
  const auto again = call(c, x, y, 100, &s1);
  const size_t bytes = want.size() * 8;
  const bool same = !std::memcmp(want.data(), got.data(), bytes) &&
                    !std::memcmp(want.data(), again.data(), bytes);
  if (s0 != CCM_OK || s1 != CCM_OK || s2 != CCM_OK || failed != 1 || !same)
    printf("status %d %d %d, %d allocations refused, results %s: %s\n", (int)s0, (int)s1, (int)s2,
           failed, same ? "the same" : "differ", ccm_last_error(c));
  else
    printf("ok\n");
  ccm_destroy(c);
  return 0;
}
