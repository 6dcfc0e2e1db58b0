// plan_report.cpp -- what the planner of libccm makes of a call, as one JSON
// line (host code only; no device is touched).
//
//   plan_report M N E,.. tau,.. L,.. r exclusion_radius query_set flags
//               [wave_limit] [walk] [spread] [max_walk_groups]
//
// missing, twice: moment slots of the results that no work item, or more than
// one, writes.  M = 0: a pair of series.  walk and spread default to the batched calls' 1.
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

// How often each moment slot is written by the plan's scans and walks.
static std::vector<int> written(const Plan& p) {
  std::vector<int> n((size_t)p.n_slots, 0);
  for (const Item& it : p.items) {
    const Realization& R = p.rz[it.rz];
    const int parts = p.shared_emax > 0 ? p.shared_emax : (p.nested.empty() ? 1 : R.n_seg);
    for (int k = 0; k < parts; ++k) ++n[(size_t)(R.slot_base + (int64_t)k * R.n_tiles + it.tile)];
  }
  for (const WalkChunk& c : p.walk_chunks)
    for (int64_t m = c.mom_first; m < c.mom_first + c.mom_count; ++m) {
      const Item& it = p.mom_items[m];
      if (!c.grouped) {
        ++n[(size_t)(p.rz[it.rz].slot_base + it.tile)];
        continue;
      }
      const WalkGroup& g = p.walk_groups[it.rz >> 2];
      const int l0 = (it.rz & 3) * kMultiLibs;
      for (int l = l0; l < std::min(g.n_lib, l0 + kMultiLibs); ++l)
        ++n[(size_t)(p.rz[p.walk_libs[g.lib_first + l].rz].slot_base + it.tile)];
    }
  return n;
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
    if (argc > 13) s.max_walk_groups = atoll(argv[13]);
    const Plan p = s.M > 0 ? make_plan_matrix(s) : make_plan(s);
    int64_t walked = 0, scanned = (int64_t)p.items.size(), spread = 0, grouped = 0, max_w = 0;
    for (char w : p.walked) walked += w != 0;
    for (const Launch& la : p.launches) spread += la.spread ? la.count : 0;
    for (const WalkChunk& c : p.walk_chunks) grouped += c.grouped ? c.mom_count : 0;
    for (const RowJob& j : p.row_jobs) max_w = std::max<int64_t>(max_w, j.w);
    int libs = 0;
    for (const WalkGroup& g : p.walk_groups) libs = std::max(libs, g.n_lib);
    // entries that placing one set's embedded points counts beforehand
    const int64_t span = query_order_span(s.N), spans = (s.N + span - 1) / span;
    int64_t missing = 0, twice = 0;
    const std::vector<int> n = written(p);
    const std::vector<Realization>& fin = p.rz_fin.empty() ? p.rz : p.rz_fin;
    for (const Realization& R : fin)
      for (int t = 0; t < R.n_tiles; ++t) {
        missing += n[(size_t)(R.slot_base + t)] == 0;
        twice += n[(size_t)(R.slot_base + t)] > 1;
      }
    printf("{\"realizations\": %zu, \"walked\": %lld, \"scan_items\": %lld, \"spread_items\": %lld, "
           "\"grouped_items\": %lld, \"groups\": %zu, \"group_libs\": %d, \"row_width\": %lld, "
           "\"out_bytes\": %lld, \"row_bytes\": %lld, \"bit_bytes\": %lld, \"mask_bytes\": %lld, "
           "\"device_bytes\": %llu, \"waves\": %zu, \"missing\": %lld, \"twice\": %lld, \"order_reads\": %lld}\n",
           p.rz.size(), (long long)walked, (long long)scanned, (long long)spread,
           (long long)grouped, p.walk_groups.size(), libs, (long long)max_w,
           (long long)p.n_walk_out * 8,
           (long long)(p.n_rows * 8 + (p.n_opts + p.n_box) * 4 +
                       p.n_todo * (int64_t)sizeof(RowTodo)),
           (long long)p.n_bits * 8, (long long)p.n_mask * 8, (unsigned long long)p.device_bytes,
           p.waves.size(), (long long)missing, (long long)twice, (long long)(spans * (spans - 1) / 2 * span));
  } catch (const Fail& e) {
    printf("{\"status\": %d}\n", (int)e.status);
    return 0;
  }
  return 0;
}
