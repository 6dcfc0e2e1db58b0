// first_call.cpp -- a call with walks that does not come again makes no graph.
// hipGraphInstantiate is taken over here to be counted.  Prints "ok" when only a
// plan's second call makes a graph and every call of it gives the same results.
#include <dlfcn.h>
#include <hip/hip_runtime_api.h>

#include <cmath>
#include <cstdio>
#include <cstring>
#include <vector>

#include "ccm.h"

static int g_graphs = 0;

extern "C" hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t g, hipGraphNode_t* n,
                                          char* log, size_t size) {
  static const auto real =
      reinterpret_cast<hipError_t (*)(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t)>(
          dlsym(RTLD_NEXT, "hipGraphInstantiate"));
  ++g_graphs;
  return real(e, g, n, log, size);
}

int main() {
  const int N = 4000, r = 100;
  const int64_t L[2] = {1000, 3000};
  std::vector<double> x(N), y(N);
  x[0] = 0.4;
  y[0] = 0.2;
  for (int t = 0; t + 1 < N; ++t) {
    x[t + 1] = x[t] * (3.8 - 3.8 * x[t] - 0.02 * y[t]);
    y[t + 1] = y[t] * (3.5 - 3.5 * y[t] - 0.1 * x[t]);
  }
  ccm_ctx* c = nullptr;
  if (ccm_create(0, &c) != CCM_OK) return 2;
  const uint64_t seeds[] = {1, 2, 3, 3, 3, 3, 4, 3};
  const int graphs[] = {0, 0, 0, 1, 1, 1, 1, 1};
  std::vector<double> first;
  int bad = 0;
  for (int k = 0; k < 8; ++k) {
    std::vector<double> rho(2 * 2 * r, -7.0);
    const ccm_status st = ccm(c, x.data(), y.data(), N, 2, 1, L, 2, r, seeds[k], nullptr,
                              rho.data(), rho.data() + 2 * r, nullptr);
    if (seeds[k] == 3 && first.empty()) first = rho;
    const bool same = seeds[k] != 3 || !std::memcmp(first.data(), rho.data(), rho.size() * 8);
    if (st != CCM_OK || g_graphs != graphs[k] || !same) {
      ++bad;
      printf("call %d: status %d, %d graphs, results %s\n", k, (int)st, g_graphs,
             same ? "the same" : "differ");
    }
  }
  if (!bad) printf("ok\n");
  ccm_destroy(c);
  return 0;
}
