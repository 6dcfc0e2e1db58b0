// plan_report.cpp -- what the planner of libccm makes of a call, as one JSON
// line (host code only; no device is touched).
//
//   plan_report M N E,.. tau,.. L,.. r exclusion_radius query_set flags
//               [wave_limit] [walk] [spread]
//
// M = 0: a pair of series.  walk and spread default to the batched calls' 1.
#include <cstdio>
#include <cstdlib>
#include <sstream>
#include <string>

#include "ccm_host.h"

using namespace ccmh;

template <class T>
static std::vector<T> list(const char* text) {
  std::vector<T> out;
  std::stringstream ss(text);
  for (std::string v; std::getline(ss, v, ',');) out.push_back((T)std::stoll(v));
  return out;
}

int main(int argc, char** argv) {
  if (argc < 10) return 2;
  const auto E = list<int32_t>(argv[3]);
  const auto tau = list<int32_t>(argv[4]);
  const auto L = list<int64_t>(argv[5]);
  ccm_opts o{atoi(argv[7]), atoi(argv[8]), (uint32_t)atoi(argv[9])};
  try {
    Spec s = make_spec(atoll(argv[2]), E.data(), (int32_t)E.size(), tau.data(),
                       (int32_t)tau.size(), L.data(), (int32_t)L.size(), atoi(argv[6]), 1, &o);
    s.M = atoi(argv[1]);
    s.wave_limit = argc > 10 ? strtoull(argv[10], nullptr, 10) : default_wave_limit(288ull << 30);
    s.walk = argc > 11 ? atoi(argv[11]) != 0 : true;
    s.spread = argc > 12 ? atoi(argv[12]) != 0 : true;
    const Plan p = s.M > 0 ? make_plan_matrix(s) : make_plan(s);
    int64_t walked = 0, scanned = (int64_t)p.items.size(), spread = 0, grouped = 0, max_w = 0;
    for (char w : p.walked) walked += w != 0;
    for (const Launch& la : p.launches) spread += la.spread ? la.count : 0;
    for (const WalkChunk& c : p.walk_chunks) grouped += c.grouped ? c.mom_count : 0;
    for (const RowJob& j : p.row_jobs) max_w = std::max<int64_t>(max_w, j.w);
    int libs = 0;
    for (const WalkGroup& g : p.walk_groups) libs = std::max(libs, g.n_lib);
    printf("{\"realizations\": %zu, \"walked\": %lld, \"scan_items\": %lld, \"spread_items\": %lld, "
           "\"grouped_items\": %lld, \"groups\": %zu, \"group_libs\": %d, \"row_width\": %lld, "
           "\"out_bytes\": %lld, \"row_bytes\": %lld, \"bit_bytes\": %lld, \"mask_bytes\": %lld, "
           "\"device_bytes\": %llu, \"waves\": %zu}\n",
           p.rz.size(), (long long)walked, (long long)scanned, (long long)spread,
           (long long)grouped, p.walk_groups.size(), libs, (long long)max_w,
           (long long)p.n_walk_out * 8,
           (long long)(p.n_rows * 8 + (p.n_opts + p.n_box) * 4 +
                       p.n_todo * (int64_t)sizeof(RowTodo)),
           (long long)p.n_bits * 8, (long long)p.n_mask * 8, (unsigned long long)p.device_bytes,
           p.waves.size());
  } catch (const Fail& e) {
    printf("{\"status\": %d}\n", (int)e.status);
    return 0;
  }
  return 0;
}
