// ccm_plan.cpp -- validation of a call and layout of its realizations,
// work items and device pools (the planner of libccm).
#include <map>
#include <numeric>
#include <unordered_map>

#include "ccm_host.h"

namespace ccmh {

OrderKey embedding_order(int32_t E, int32_t tau) {
  if (E == 1) return {1, {0, 0, 0, 0}};
#ifndef CCM_KD_MIN_E
#define CCM_KD_MIN_E 3
#endif
  if (E < CCM_KD_MIN_E) return {2, {0, tau, 0, 0}};
  // sorted first on the newest coordinate, which puts exactly the embedded
  // points (i < n_e) first; the k-d levels then reorder them
  return {1, {(E - 1) * tau, 0, 0, 0}, E};
}

// Leaves of about this many points end the k-d refinement.
#ifndef CCM_KD_LEAF
#define CCM_KD_LEAF 48
#endif
constexpr int64_t kKdLeaf = CCM_KD_LEAF;
constexpr int kKdMaxLevels = 12;

void attach_kd(Plan& p, int64_t key_off, int32_t E, int64_t emb_off, int64_t ne) {
  OrderJob& o = p.orders[(size_t)(key_off / p.spec.N)];
  if (o.kd_E == 0) return;
  o.kd_emb_off = emb_off;
  o.kd_n_e = ne;
  int lv = 1;
  while (lv < kKdMaxLevels && (ne >> lv) > kKdLeaf) ++lv;
  o.kd_levels = lv;
  p.kd_levels = std::max(p.kd_levels, lv);
  if (!p.embed.empty()) p.embed.back().whole = 1;
  (void)E;
}

OrderKey shared_order(int32_t Emax, int32_t tau) {
  if (Emax == 1) return {1, {0, 0, 0, 0}};
  if (Emax < 6) return {2, {(Emax - 2) * tau, (Emax - 1) * tau, 0, 0}};
  return {4, {(Emax - 1) * tau, (Emax - 2) * tau, (Emax - 3) * tau, (Emax - 4) * tau}};
}

int64_t order_set(Plan& p, int series, const OrderKey& key) {
  const int64_t N = p.spec.N;
  for (size_t k = 0; k < p.orders.size(); ++k) {
    const OrderJob& o = p.orders[k];
    if (o.src_off == series * N && o.dims == key.dims && o.kd_E == key.kd_E &&
        std::equal(key.lag, key.lag + 4, o.lag))
      return o.key_off;
  }
  const int64_t off = (int64_t)p.orders.size() * N;
  OrderJob o{};
  o.src_off = series * N;
  o.key_off = off;
  o.n = N;
  o.dims = key.dims;
  for (int d = 0; d < 4; ++d) o.lag[d] = key.lag[d];
  o.kd_E = key.kd_E;
  p.orders.push_back(o);
  p.n_sets = (int32_t)p.orders.size();
  p.n_ord = p.n_sets * N;
  if (p.n_ord > (int64_t)INT32_MAX) fail(CCM_E_INVAL, "too many time points to order");
  return off;
}

// A realization walks a table when the flag asks for it, its embedding fits
// the walk's LDS bitmask, the expected walk to E+1 acceptable library members
// ((E+1+excluded) n_e / l_eff row entries) is at most a quarter of a
// truncated row (a wavefront whose walk runs short scans instead, which must
// stay rare), and the walk (about 8 instructions per entry) is cheaper than
// the scan (2E per pair).
bool use_table(const Plan& p, int E, int64_t ne, int64_t le) {
  if (!(p.spec.flags & CCM_FLAG_TABLE) || ne > kTableMaxNe) return false;
  const double excl =
      p.mode == kExclSelf ? 1.0 : (p.mode == kWindow ? 2.0 * p.window + 1.0 : 0.0);
  const double walk = (E + 1 + excl) * (double)ne / (double)le;
  const int64_t w = std::min<int64_t>(kTableWidth, ne);
  if (w < ne && walk > (double)w / 4.0) return false;
  return 8.0 * walk < 2.0 * E * (double)le;
}

int64_t table_for(Plan& p, int64_t emb_off, int64_t ne, int E) {
  for (const TableJob& t : p.tables)
    if (t.emb_off == emb_off) return t.out_off;
  const int32_t w = (int32_t)std::min<int64_t>(kTableWidth, ne);
  TableJob t{};
  t.emb_off = emb_off;
  t.out_off = p.n_table;
  t.n_e = (int32_t)ne;
  t.E = E;
  t.w = w;
  if (p.te_count[E] == 0) p.te_first[E] = (int)p.tables.size();
  p.te_count[E] += 1;
  p.te_max_ne[E] = std::max(p.te_max_ne[E], (int)ne);
  p.tables.push_back(t);
  p.n_table += ne * table_row_stride(w);
  return t.out_off;
}

uint64_t default_wave_limit(uint64_t total) {
  return std::max<uint64_t>(1ull << 30, std::min<uint64_t>(8ull << 30, total / 8));
}

// Pool bytes of one realization in its wave: its gathered library (binary32
// coordinates and int32 indices), and, once per wave, its library draw (a
// nested shuffle also keeps its n_e positions).
static uint64_t draw_bytes(const Plan& p, int64_t sj) {
  if (!p.nested.empty()) return ((uint64_t)p.nested[sj].n_out + (uint64_t)p.nested[sj].n_e) * 4;
  return (uint64_t)p.sample[sj].l_eff * 4;
}
static uint64_t points_bytes(const Realization& R) {
  return (uint64_t)R.l_eff * (uint64_t)(R.E + 1) * 4;
}

// Group the realizations into waves whose pools fit spec.wave_limit (0: one
// wave): all realizations of one E together when they fit, consecutive E
// merged while they fit, an E too large for one wave split into several.
// Then lay out each wave's draws and gathered libraries from offset 0 of
// the shared pools (a draw used by realizations of two waves is drawn in
// both) and rebase the realizations and jobs that refer to them.
static void split_waves(Plan& p) {
  const uint64_t limit = p.spec.wave_limit;
  const bool nested = !p.nested.empty();
  const size_t n = p.rz.size();
  std::vector<int32_t> order(n);
  std::iota(order.begin(), order.end(), 0);
  std::stable_sort(order.begin(), order.end(),
                   [&](int32_t a, int32_t b) { return p.rz[a].E < p.rz[b].E; });

  std::vector<std::vector<int32_t>> waves;
  std::vector<int32_t> cur;
  std::unordered_map<int64_t, int> cur_draws;
  uint64_t cur_b = 0;
  auto close_wave = [&] {
    if (!cur.empty()) waves.push_back(std::move(cur));
    cur.clear();
    cur_draws.clear();
    cur_b = 0;
  };
  auto add = [&](int32_t r) {
    cur.push_back(r);
    cur_b += points_bytes(p.rz[r]);
    if (cur_draws.emplace(p.rz_sample[r], 1).second) cur_b += draw_bytes(p, p.rz_sample[r]);
  };
  for (size_t g0 = 0; g0 < n;) {
    size_t g1 = g0;
    while (g1 < n && p.rz[order[g1]].E == p.rz[order[g0]].E) ++g1;
    // bytes of the whole E group (its draws counted once each)
    uint64_t gb = 0;
    {
      std::unordered_map<int64_t, int> d;
      for (size_t k = g0; k < g1; ++k) {
        gb += points_bytes(p.rz[order[k]]);
        if (d.emplace(p.rz_sample[order[k]], 1).second) gb += draw_bytes(p, p.rz_sample[order[k]]);
      }
    }
    if (limit == 0 || cur_b + gb <= limit) {
      for (size_t k = g0; k < g1; ++k) add(order[k]);
    } else if (gb <= limit) {
      close_wave();
      for (size_t k = g0; k < g1; ++k) add(order[k]);
    } else {
      close_wave();
      for (size_t k = g0; k < g1; ++k) {
        const int32_t r = order[k];
        uint64_t b = points_bytes(p.rz[r]);
        if (!cur_draws.count(p.rz_sample[r])) b += draw_bytes(p, p.rz_sample[r]);
        if (!cur.empty() && cur_b + b > limit) close_wave();
        add(r);
      }
    }
    g0 = g1;
  }
  close_wave();

  std::vector<SampleJob> sample;
  std::vector<NestedJob> shuffles;
  std::vector<GatherJob> gather;
  int64_t max_lib = 0, max_pts = 0, max_pj = 0, max_scr = 0;
  p.waves.clear();
  p.wave_rz.clear();
  p.wave_rz_first.clear();
  for (const auto& wr : waves) {
    Wave w;
    w.sample_first = nested ? (int64_t)shuffles.size() : (int64_t)sample.size();
    w.gather_first = (int64_t)gather.size();
    p.wave_rz_first.push_back((int64_t)p.wave_rz.size());
    std::unordered_map<int64_t, int64_t> remap;   // draw: old index -> new index
    int64_t lib = 0, pts = 0, pj = 0, scr = 0;
    for (int32_t r : wr) {
      p.wave_rz.push_back(r);
      const int64_t sj = p.rz_sample[r];
      int64_t old_out = 0, new_out = 0;
      auto it = remap.find(sj);
      if (nested) {
        old_out = p.nested[sj].out_off;
        if (it == remap.end()) {
          NestedJob j = p.nested[sj];
          j.out_off = lib;
          j.scratch_off = scr;
          lib += j.n_out;
          scr += j.n_e;
          it = remap.emplace(sj, (int64_t)shuffles.size()).first;
          shuffles.push_back(j);
        }
        new_out = shuffles[it->second].out_off;
      } else {
        old_out = p.sample[sj].out_off;
        if (it == remap.end()) {
          SampleJob j = p.sample[sj];
          j.out_off = lib;
          lib += j.l_eff;
          it = remap.emplace(sj, (int64_t)sample.size()).first;
          sample.push_back(j);
        }
        new_out = sample[it->second].out_off;
      }
      Realization& R = p.rz[r];
      const int64_t ng = nested ? R.n_seg : 1;
      const int64_t g0 = p.rz_gather[r];
      p.rz_gather[r] = (int64_t)gather.size();
      for (int64_t g = g0; g < g0 + ng; ++g) {
        GatherJob G = p.gather[g];
        G.lib_off = new_out + (G.lib_off - old_out);
        G.pts_off = pts + (G.pts_off - R.pts_off);
        G.pj_off = pj + (G.pj_off - R.pj_off);
        if (G.sorted) w.max_sorted_n_e = std::max(w.max_sorted_n_e, G.n_e);
        gather.push_back(G);
      }
      p.rz_sample[r] = it->second;
      R.pts_off = pts;
      R.pj_off = pj;
      pts += (int64_t)R.l_eff * R.E;
      pj += R.l_eff;
    }
    w.sample_count = (nested ? (int64_t)shuffles.size() : (int64_t)sample.size()) - w.sample_first;
    w.gather_count = (int64_t)gather.size() - w.gather_first;
    w.pool_bytes = (uint64_t)(lib + pj + scr) * 4 + (uint64_t)pts * 4;
    p.waves.push_back(w);
    max_lib = std::max(max_lib, lib);
    max_pts = std::max(max_pts, pts);
    max_pj = std::max(max_pj, pj);
    max_scr = std::max(max_scr, scr);
  }
  p.wave_rz_first.push_back((int64_t)p.wave_rz.size());
  if (nested)
    p.nested = std::move(shuffles);
  else
    p.sample = std::move(sample);
  p.gather = std::move(gather);
  p.n_lib = max_lib;
  p.n_pts = max_pts;
  p.n_pj = max_pj;
  if (nested) p.n_scratch = max_scr;
}

// Device bytes of neighbour rows held at once (a batch holds at least one
// embedding's; a single embedding past the cap scans instead), and of walk
// output held at once: predictions (256 MiB was 1% slower, 1 GiB the same), or
// a causal matrix's neighbour keys (its per-target stage has few, long items:
// 512 MiB 21.9 against 18.4 ms for 64 series, N = 20000, r = 10).  A group of
// 64 libraries whose output is larger by itself (pairs beyond 2^20 points, a
// matrix beyond 2^21 / (E+1)) is made of fewer.
constexpr int64_t kRowPoolBytes = 1ll << 30;
constexpr int64_t kRowPoolCap = 2ll << 30;
constexpr int64_t kWalkOutBytes = 512ll << 20;
constexpr int64_t kWalkKeyBytes = 1ll << 30;
constexpr int64_t kMultiMinItems = 1024;
// Launches of scans that spread their queries over more wavefronts: at most
// two wavefronts per SIMD otherwise, and a serial scan that outweighs the
// second launch's 6 us, in instructions per lane (198 libraries of a pair of 777
// points, up to 770 at E = 3: scan 122 us, spread 40 + 7; 119 points at E = 2:
// 27 and 10 + 6; 46 to 87 points: calls 5 to 10 us longer).  Beside walks the
// scan is not what the call waits for (5003 points at E = 7: 543 and 556 us).
constexpr int32_t kSpreadItems = 512;
constexpr double kSpreadMinWork = 2500.0;

// Row entries that hold, all but about once in 10^7, the first E+1 acceptable
// members of a library of le of ne points: a member turns up every ne / le
// entries, and the spread of their number is at most a Poisson variable's;
// `excl` entries may be excluded ones.  (At once in 10^5 the searches of the
// libraries that ran short took longer than the rest of the walk at N = 10^5,
// 5.0 against 1.1 ms.)
static int64_t row_need(int E, double excl, int64_t ne, int64_t le) {
  const double k = E + 1;
  const double n = (k + 5.5 * std::sqrt(k) + 9.0) * (double)ne / (double)le + excl;
  return n < 1e9 ? (int64_t)n + 1 : (int64_t)1e9;
}

// Libraries of an embedding of ne points that walk together.  (Nested and
// shared-E calls walk up to 2^18 points at most, where 64 always fit.)
static size_t group_libs(const Plan& p, int E, int64_t ne) {
  const int64_t each = p.spec.M > 0 ? ne * (E + 1) * 8 : ne * 8;
  const int64_t bytes = p.spec.M > 0 ? kWalkKeyBytes : kWalkOutBytes;
  return (size_t)std::max<int64_t>(1, std::min<int64_t>(kWalkLibs, bytes / each));
}

// Costs in instruction slots of a wavefront, per query of an embedding: one
// scanned library (64 queries share a wavefront), one walk of a group of
// libraries, and building a row of w entries.
static double scan_cost(int E, int64_t le) {
  return ((2.0 * E + 4.0) * (double)le * 1.25 + 110.0 * (E + 1) + 120.0) / 64.0;
}
static double walk_cost(int E, int64_t chunks) {
  return 150.0 + 150.0 * (double)chunks + 30.0 * (E + 1) + 90.0 * (E + 1);
}
static double row_cost(int E, int64_t ne, int64_t w) {
  return (2.0 * E + 20.0) * (double)ne / 64.0 + 8.0 * (double)w + 1500.0;
}
// Slots below which the walk's seven launches cost more than it saves (at
// 2 x 10^7 a pair of N = 1331 at E = 1 went from 153 to 183 us).
constexpr double kWalkMinGain = 5.0e7;

// Long series in many dimensions: a row's pass visits the runs of 64 points that
// the ball of its nearest 1.5 w reaches, and the costs above hold for points on
// an attractor of few dimensions.  Points that fill theirs (shuffled series)
// take a multiple: about (0.7 (1.5 w)^(1/E) + 64^(1/E))^E / 64 runs, up to all.
// `scan` and `walk`: nanoseconds of the whole chip per query, as below; a scan of
// few items leaves part of its last round of workgroups (1536 resident) idle.
// True where shuffled series would take over 1.45 times as long as scanned, and
// so longer than before there were rows: 32768 points, E = 9, 40 libraries of
// 2048, 10.1 ms walked, 3.5 scanned, 5.2 then (in the logistic map's order 3.4, 3.1
// and 4.8); 10^5 points, 40 of 6250, 28.9, 20.2 and 24.4 (9.1, 19.1 and 23.4).
// Below E = 7, and below 20000 points, shuffled series took less than then.
static bool rows_too_dear(int E, int64_t ne, int64_t w, double scan, double walk, int64_t items) {
  if (E < 7 || ne < 20000) return false;
  const double side = 0.7 * std::pow(1.5 * (double)w, 1.0 / E) + std::pow(64.0, 1.0 / E);
  const double runs = std::min((double)ne / 64.0, std::pow(side, E) / 64.0);
  const double rows = 3.0 + 0.0024 * E * (double)w + 0.25 * runs + 6.8e-6 * E * (double)ne;
  const double rounds = std::ceil((double)items / 1536.0) * 1536.0 / (double)items;
  return 1.45 * rounds * scan < walk + rows;
}
// A scanned library, and a walk of a group (pairs of 10^4 to 10^5 points, E = 1 to
// 10: within a factor 1.3).
static double scan_ns(int E, int64_t le) {
  return 0.042 + 3.2e-5 * E * (double)le + 0.0015 * E * std::log2((double)std::max<int64_t>(le, 1));
}
static double walk_ns(int E, int64_t chunks) {
  return 0.74 + 0.12 * E + 0.27 * (double)chunks;
}

// Causal matrices of more than 8 series: the same by query of an embedding.  A walk
// leaves keys to a per-target stage of its own, which takes longer than the stage
// within the scan (M = 17, N = 2050, E = 5, 64 libraries: 5.6 x 10^3 by this count,
// 1.86 ms walked, 1.17 scanned, 1.44 before there were rows; M = 17, N = 9284, E = 7: 2
// x 10^4, 5.1 and 6.1).  Of 23 calls below 8000, 20 were faster scanned, by 1.08 to
// 1.75 times, the others slower by 1.05 to 1.24.
constexpr double kMatrixMinGain = 8000.0;

// Groups of one embedding's libraries that walk its rows together.
struct WalkPick {
  std::vector<std::vector<int32_t>> groups;
  std::vector<int32_t> chunks;      // 64-entry chunks each group may need
  int64_t w = 0;
};

// The libraries of one embedding (v: its realizations in one launch) worth
// walking: the largest first, in groups, as many groups as each save
// more than they cost.  Returns the slots saved per query, the rows' cost
// not counted; forced: CCM_FLAG_TABLE asks for some of them.
static double pick_libraries(const Plan& p, int E, double excl, std::vector<int32_t>& v,
                             int64_t n_emb, WalkPick& pk, bool& forced) {
  std::stable_sort(v.begin(), v.end(), [&](int32_t a, int32_t b) {
    const bool fa = p.want_table[a] != 0, fb = p.want_table[b] != 0;
    if (fa != fb) return fa;
    return p.rz[a].l_eff > p.rz[b].l_eff;
  });
  const int64_t ne = p.rz[v[0]].n_e;
  const int64_t full = (ne + 63) / 64 * 64;
  const size_t libs = group_libs(p, E, ne);
  double gain = 0, all_scan = 0, all_walk = 0;
  int64_t items = 0;                // of the scans, every embedding's
  const auto row_width = [&](int32_t r) {
    return std::min(full, (row_need(E, excl, ne, p.rz[r].l_eff) + 63) / 64 * 64);
  };
  for (size_t g0 = 0; g0 < v.size(); g0 += libs) {
    const size_t g1 = std::min(v.size(), g0 + libs);
    std::vector<int32_t> grp;
    bool force = false;
    for (size_t k = g0; k < g1; ++k) {
      const bool want = p.want_table[v[k]] != 0;
      if (row_width(v[k]) > kRowMaxW && !want) continue;
      force |= want;
      grp.push_back(v[k]);
    }
    // Library-point queries: a small library asks few of the rows that it
    // lengthens for all, so the group ends where it saves most (70 series of 17687
    // points, E = 1, libraries of 11036 to 14815 points and of 337 to 556: rows of
    // 1024 entries 21.8 ms, 19.0 before there were rows; of 64, 10.7).
    const bool cut = p.spec.query_set != 0 && !force;
    const double rows0 = row_cost(E, ne, pk.groups.empty() ? 64 : pk.w);
    double scan = 0, ns = 0, sum = 0, sum_ns = 0, most = 0;
    int64_t need = 64, tiles = 0, sum_tiles = 0, width = 64;
    size_t keep = 0;
    for (size_t k = 0; k < grp.size(); ++k) {
      const Realization& R = p.rz[grp[k]];
      const double asked = (double)R.n_query / (double)ne;
      sum += scan_cost(E, R.l_eff) * asked;
      sum_ns += scan_ns(E, R.l_eff) * asked;
      sum_tiles += R.n_tiles;
      width = std::max(width, std::min<int64_t>(row_width(grp[k]), kRowMaxW));
      const double net = sum - walk_cost(E, width / 64) -
                         (row_cost(E, ne, std::max(pk.w, width)) - rows0);
      if (cut && net <= most) continue;
      most = net;
      keep = k + 1;
      scan = sum;
      ns = sum_ns;
      tiles = sum_tiles;
      need = width;
    }
    grp.resize(keep);
    if (grp.empty()) continue;
    const double save = scan - walk_cost(E, need / 64);
    if (save <= 0 && !force) continue;
    gain += save;
    all_scan += ns;
    items += tiles * n_emb;
    all_walk += walk_ns(E, need / 64);
    forced |= force;
    pk.w = std::max(pk.w, need);
    pk.groups.push_back(std::move(grp));
    pk.chunks.push_back((int32_t)(need / 64));
  }
  return rows_too_dear(E, ne, pk.w, all_scan, all_walk, items) ? 0.0 : gain;
}

// The same for nested libraries (v: the embedding's chains): a chain's scan
// reads each segment once for every size after it, so the sizes that walk are
// the last ones of every chain, from the size `first` on which saves most.
// Each becomes a realization of its own (appended to p.rz; slots as the
// chain's), and the chains keep the segments before it.  Row widths as above.
static double pick_sizes(const Plan& p, int E, double excl, const std::vector<int32_t>& v,
                         int64_t n_emb, int& first) {
  const Realization& R = p.rz[v[0]];
  const int64_t ne = R.n_e;
  const int64_t full = (ne + 63) / 64 * 64;
  const int32_t* seg = &p.segs[R.seg_off];
  const double n = (double)v.size();
  double best = 0, walk = 0, ns = 0;
  first = R.n_seg;
  for (int k = R.n_seg - 1; k >= 0; --k) {
    const int64_t w = std::min(full, (row_need(E, excl, ne, seg[k + 1]) + 63) / 64 * 64);
    if (w > kRowMaxW) break;
    walk += walk_cost(E, w / 64) * n / kWalkLibs;
    ns += walk_ns(E, w / 64) * n / kWalkLibs;
    const double saved = n * (scan_ns(E, R.l_eff) - scan_ns(E, seg[k]) +
                              (double)(R.n_seg - k) * scan_ns(E, 0));
    if (rows_too_dear(E, ne, w, saved, ns, (int64_t)v.size() * n_emb * R.n_tiles)) continue;
    // what the chains' scans lose: the points past seg[k], one selection and
    // prediction per size
    const double scan = n * (scan_cost(E, R.l_eff) - scan_cost(E, seg[k]) +
                             (double)(R.n_seg - 1 - k) * scan_cost(E, 0) +
                             (k == 0 ? scan_cost(E, 0) : 0.0));
    const double gain = scan - walk - row_cost(E, ne, w);
    if (gain > best) {
      best = gain;
      first = k;
    }
  }
  return best;
}

// A realization of its own for a library walked out of realization `of`
// (same draw and gather jobs); returns its index.
static int32_t add_walked(Plan& p, const Realization& R, int32_t of) {
  if (p.rz.size() >= (size_t)INT32_MAX) fail(CCM_E_INVAL, "too many realizations");
  p.rz.push_back(R);
  p.rz_sample.push_back((int64_t)p.rz_sample[of]);
  p.rz_gather.push_back((int64_t)p.rz_gather[of]);
  p.want_table.push_back(0);
  p.walked.push_back(1);
  p.walk_out.push_back(WalkOut{});
  return (int32_t)p.rz.size() - 1;
}

static void nested_libraries(Plan& p, int E, double excl, const std::vector<int32_t>& v, int first,
                             WalkPick& pk) {
  std::vector<int32_t> libs;
  const int n_seg = p.rz[v[0]].n_seg;
  for (int k = n_seg - 1; k >= first; --k)
    for (int32_t chain : v) {
      Realization R = p.rz[chain];
      R.l_eff = p.segs[R.seg_off + k + 1];
      R.slot_base += (int64_t)k * R.n_tiles;
      R.n_seg = 0;
      R.seg_off = k;                // (the size: for its bitmap)
      libs.push_back(add_walked(p, R, chain));
    }
  for (int32_t chain : v) {
    p.rz[chain].n_seg = first;
    NestedJob& nj = p.nested[p.rz_sample[chain]];
    nj.seg0 = std::min(nj.bits ? nj.seg0 : n_seg, first);
    nj.bits = -1;                   // placed by the caller
  }
  const int64_t ne = p.rz[v[0]].n_e;
  const int64_t full = (ne + 63) / 64 * 64;
  for (size_t g0 = 0; g0 < libs.size(); g0 += kWalkLibs) {
    const size_t g1 = std::min(libs.size(), g0 + kWalkLibs);
    // sizes fall: the last library needs the longest row
    const int64_t le = p.rz[libs[g1 - 1]].l_eff;
    const int64_t w = std::min(full, (row_need(E, excl, ne, le) + 63) / 64 * 64);
    pk.w = std::max(pk.w, w);
    pk.groups.emplace_back(libs.begin() + g0, libs.begin() + g1);
    pk.chunks.push_back((int32_t)(w / 64));
  }
}

// Whether the plan can number `more` walk groups.
static bool groups_fit(const Plan& p, size_t more) {
  return (int64_t)(p.walk_groups.size() + more) <= p.spec.max_walk_groups;
}

// Lay out the walks of one launch: per pick (an embedding's groups) a row
// job, the groups' libraries, bitmaps and membership words, the batches of
// embeddings whose rows fit together and the chunks whose output does.
static void lay_out_walks(Plan& p, std::vector<WalkPick>& picks, Launch& la, int64_t& bits) {
  const int E = la.E;
  const bool keys = p.spec.M > 0;
  const bool nested = !p.nested.empty();
  // groups of different embeddings that draw the same libraries share masks
  std::map<std::vector<int64_t>, int64_t> mask_of;
  int64_t masks = 0, total_q = 0;
  la.mask_first = (int32_t)p.mask_jobs.size();
  std::vector<size_t> emb_group;      // first group of each row job
  const int32_t job0 = (int32_t)p.row_jobs.size();
  for (WalkPick& pk : picks) {
    const Realization& R0 = p.rz[pk.groups[0][0]];
    RowJob rj{};
    rj.emb_off = R0.emb_off;
    rj.qord_off = R0.qord_off;
    rj.n_e = R0.n_e;
    rj.w = (int32_t)pk.w;
    rj.stride = p.shared_emax > 0 ? p.shared_emax : E;
    emb_group.push_back(p.walk_groups.size());
    for (size_t g = 0; g < pk.groups.size(); ++g) {
      const std::vector<int32_t>& grp = pk.groups[g];
      WalkGroup wg{};
      wg.lib_first = (int64_t)p.walk_libs.size();
      wg.tgt_off = keys ? 0 : R0.tgt_off + (int64_t)(E - 1) * R0.tau;
      wg.n_lib = (int32_t)grp.size();
      wg.emb = (int32_t)p.row_jobs.size();
      wg.chunks = pk.chunks[g];
      std::vector<int64_t> sig;
      for (int32_t r : grp) {
        WalkLib wl{};
        // the draw's bitmap, one per draw of the wave
        if (nested) {
          const NestedJob& nj = p.nested[p.rz_sample[r]];
          wl.bit_off = nj.bits - 1 + (p.rz[r].seg_off - nj.seg0) * ((nj.n_e + 63) / 64);
        } else {
          SampleJob& sj = p.sample[p.rz_sample[r]];
          if (sj.bits == 0) {
            sj.bits = 1 + bits;
            bits += (sj.n_e + 63) / 64;
          }
          wl.bit_off = sj.bits - 1;
        }
        wl.rz = r;
        p.walk_libs.push_back(wl);
        p.walked[r] = 1;
        if (p.want_table[r]) p.table_rz += keys ? p.spec.M - 1 : 1;
        sig.push_back(wl.bit_off);
      }
      const auto it = mask_of.emplace(sig, masks);
      wg.mask_off = it.first->second;
      if (it.second) {
        p.mask_jobs.push_back({masks, wg.lib_first, wg.n_lib, rj.n_e});
        la.mask_max_ne = std::max(la.mask_max_ne, rj.n_e);
        masks += rj.n_e;
      }
      p.walk_groups.push_back(wg);
      total_q += rj.n_e;
    }
    p.row_jobs.push_back(rj);
  }
  emb_group.push_back(p.walk_groups.size());
  la.mask_count = (int32_t)p.mask_jobs.size() - la.mask_first;
  p.n_mask = std::max(p.n_mask, masks);

  // enough items to fill the chip, at most 64 queries each
  la.walk_per = (int32_t)std::min<int64_t>(64, std::max<int64_t>(4, total_q / 8192 / 4 * 4));

  la.batch_first = (int32_t)p.walk_batches.size();
  const int32_t n_jobs = (int32_t)p.row_jobs.size() - job0;
  const int64_t per_query = keys ? E + 1 : 1;
  for (int32_t e0 = 0; e0 < n_jobs;) {
    WalkBatch wb;
    wb.emb_first = job0 + e0;
    int64_t rows = 0, opts = 0, box = 0, n_row = 0;
    int32_t e1 = e0;
    for (; e1 < n_jobs; ++e1) {
      RowJob& rj = p.row_jobs[job0 + e1];
      const int64_t need = (int64_t)rj.n_e * rj.w;
      if (e1 > e0 && (rows + need) * 8 > kRowPoolBytes) break;
      if (e1 - e0 >= 65535) break;
      rj.out_off = rows;
      rj.pts_off = opts;
      rj.box_off = box;
      rows += need;
      opts += (int64_t)rj.n_e * E;
      box += (int64_t)((rj.n_e + 64 * 256 - 1) / (64 * 256)) * 256 * 2 * E;
      n_row += rj.n_e;
      wb.max_ne = std::max(wb.max_ne, rj.n_e);
      wb.max_w = std::max(wb.max_w, rj.w);
    }
    wb.emb_count = e1 - e0;
    wb.rows_per_block = (int32_t)std::min<int64_t>(16, std::max<int64_t>(1, n_row / 4096));
    p.n_rows = std::max(p.n_rows, rows);
    p.n_opts = std::max(p.n_opts, opts);
    p.n_box = std::max(p.n_box, box);
    p.n_todo = std::max(p.n_todo, n_row);
    wb.chunk_first = (int32_t)p.walk_chunks.size();
    // chunks: consecutive groups whose output fits; within a chunk the
    // groups of one embedding take the same block of queries together, so
    // they read its rows from cache
    size_t g = emb_group[e0];
    const size_t g_end = emb_group[e1];
    while (g < g_end) {
      WalkChunk ch;
      ch.item_first = (int64_t)p.walk_items.size();
      ch.mom_first = (int64_t)p.mom_items.size();
      int64_t out = 0;
      size_t h = g;
      for (; h < g_end; ++h) {
        WalkGroup& wg = p.walk_groups[h];
        // whole cache lines per group
        const int64_t need =
            ((int64_t)wg.n_lib * p.row_jobs[wg.emb].n_e * per_query + 15) / 16 * 16;
        if (h > g && (out + need) * 8 > (keys ? kWalkKeyBytes : kWalkOutBytes)) break;
        wg.out_off = out;
        for (int l = 0; l < wg.n_lib; ++l)
          p.walk_out[p.walk_libs[wg.lib_first + l].rz] = {out + l, wg.n_lib, 0};
        out += need;
      }
      // causal matrix over every point: kMultiLibs libraries to an item when
      // that leaves enough items (3 series, N = 5809: 54 items took 1.9 ms, one
      // per library 1.3 ms)
      int64_t parts = 0;
      for (size_t x = g; x < h; ++x)
        parts += (int64_t)((p.walk_groups[x].n_lib + kMultiLibs - 1) / kMultiLibs) *
                 p.rz[p.walk_libs[p.walk_groups[x].lib_first].rz].n_tiles;
      ch.grouped = keys && p.spec.query_set == 0 && parts >= kMultiMinItems;
      for (size_t a = g; a < h;) {
        size_t b = a;
        while (b < h && p.walk_groups[b].emb == p.walk_groups[a].emb) ++b;
        const int32_t ne = p.row_jobs[p.walk_groups[a].emb].n_e;
        const int32_t blocks = (ne + la.walk_per - 1) / la.walk_per;
        for (int32_t q = 0; q < blocks; ++q)
          for (size_t x = a; x < b; ++x) p.walk_items.push_back({(int32_t)x, q});
        // a tile of every library of a group together: they read the same
        // cache lines of the walk's output (and the same target rows)
        for (size_t x = a; x < b; ++x) {
          const WalkGroup& wg = p.walk_groups[x];
          int32_t tiles = 0;
          for (int l = 0; l < wg.n_lib; ++l)
            tiles = std::max(tiles, p.rz[p.walk_libs[wg.lib_first + l].rz].n_tiles);
          if (ch.grouped) {
            for (int32_t t = 0; t < tiles; ++t)
              for (int l = 0; l < wg.n_lib; l += kMultiLibs)
                p.mom_items.push_back({(int32_t)(4 * x) + l / kMultiLibs, t});
            continue;
          }
          for (int32_t t = 0; t < tiles; ++t)
            for (int l = 0; l < wg.n_lib; ++l) {
              const int32_t r = p.walk_libs[wg.lib_first + l].rz;
              if (t < p.rz[r].n_tiles) p.mom_items.push_back({r, t});
            }
        }
        a = b;
      }
      ch.item_count = (int64_t)p.walk_items.size() - ch.item_first;
      ch.mom_count = (int64_t)p.mom_items.size() - ch.mom_first;
      p.n_walk_out = std::max(p.n_walk_out, out);
      p.walk_chunks.push_back(ch);
      g = h;
    }
    wb.chunk_count = (int32_t)p.walk_chunks.size() - wb.chunk_first;
    p.walk_batches.push_back(wb);
    e0 = e1;
  }
  la.batch_count = (int32_t)p.walk_batches.size() - la.batch_first;
}

// The realizations of one launch (rzs: one E of one wave) that walk
// neighbour rows: per embedding those picked above, when all they save
// together exceeds the cost of the rows and launches.
static void plan_walks(Plan& p, const std::vector<int32_t>& rzs, Launch& la, int64_t& bits) {
  if (!p.spec.walk || rzs.empty()) return;
  const int E = la.E;
  const bool nested = !p.nested.empty();
  // the shuffle's bitmaps come from positions in LDS
  if (nested && p.spec.N > kNestedLdsNe) return;
  const double excl =
      p.mode == kExclSelf ? 1.0 : (p.mode == kWindow ? 2.0 * p.window + 1.0 : 0.0);
  std::map<int64_t, std::vector<int32_t>> by_emb;   // in embedding order
  for (int32_t r : rzs) by_emb[p.rz[r].emb_off].push_back(r);

  std::vector<WalkPick> picks;
  double gain_all = 0;
  bool forced_any = false;
  if (nested) {
    std::vector<std::pair<const std::vector<int32_t>*, int>> sizes;
    size_t groups = 0;
    for (auto& kv : by_emb) {
      int first = 0;
      const double gain = pick_sizes(p, E, excl, kv.second, (int64_t)by_emb.size(), first);
      const Realization& R = p.rz[kv.second[0]];
      if (gain <= 0 || (int64_t)R.n_e * kRowMaxW * 8 > kRowPoolCap) continue;
      gain_all += gain * (double)R.n_e;
      groups += kv.second.size() * (size_t)(R.n_seg - first) / kWalkLibs + 1;
      sizes.emplace_back(&kv.second, first);
    }
    if (gain_all < kWalkMinGain || !groups_fit(p, groups)) return;
    for (auto& s : sizes) {
      picks.emplace_back();
      nested_libraries(p, E, excl, *s.first, s.second, picks.back());
    }
    for (auto& s : sizes)
      for (int32_t chain : *s.first) {
        NestedJob& nj = p.nested[p.rz_sample[chain]];
        if (nj.bits >= 0) continue;               // placed already
        nj.bits = 1 + bits;
        bits += (int64_t)(nj.n_seg - nj.seg0) * ((nj.n_e + 63) / 64);
      }
  } else {
    size_t groups = 0;
    double queries = 0;
    for (auto& kv : by_emb) {
      WalkPick pk;
      bool forced = false;
      double gain = pick_libraries(p, E, excl, kv.second, (int64_t)by_emb.size(), pk, forced);
      const int64_t ne = p.rz[kv.second[0]].n_e;
      const bool fits = ne * pk.w * 8 <= kRowPoolCap;
      gain = (gain - row_cost(E, ne, pk.w)) * (double)ne;
      if (pk.groups.empty() || !fits || (gain <= 0 && !forced)) continue;
      gain_all += gain;
      forced_any |= forced;
      groups += pk.groups.size();
      queries += (double)ne;
      picks.push_back(std::move(pk));
    }
    if (p.spec.M > 8 && !forced_any && gain_all < kMatrixMinGain * queries) return;
    if (picks.empty() || (gain_all < kWalkMinGain && !forced_any) || !groups_fit(p, groups)) return;
  }
  if (!picks.empty()) lay_out_walks(p, picks, la, bits);
}

// E-sweep sharing: realizations (scans of every E at once) whose libraries
// walk the rows of each requested E instead, over the first E coordinates of
// the shared embedding: one walked realization per E, in the scan's slots.
static void plan_shared_walks(Plan& p, const std::vector<int32_t>& rzs, Launch& la,
                              int64_t& bits) {
  if (!p.spec.walk || rzs.empty()) return;
  const int Emax = p.shared_emax;
  const double excl =
      p.mode == kExclSelf ? 1.0 : (p.mode == kWindow ? 2.0 * p.window + 1.0 : 0.0);
  std::vector<int32_t> Es = p.spec.E;
  std::sort(Es.begin(), Es.end());
  Es.erase(std::unique(Es.begin(), Es.end()), Es.end());
  std::map<int64_t, std::vector<int32_t>> by_emb;
  for (int32_t r : rzs) by_emb[p.rz[r].emb_off].push_back(r);

  std::vector<std::vector<std::vector<int32_t>>> groups;   // per embedding
  size_t n_groups = 0;
  double gain_all = 0;
  for (auto& kv : by_emb) {
    std::vector<int32_t>& v = kv.second;
    std::stable_sort(v.begin(), v.end(),
                     [&](int32_t a, int32_t b) { return p.rz[a].l_eff > p.rz[b].l_eff; });
    const int64_t ne = p.rz[v[0]].n_e;
    if (ne * kRowMaxW * 8 > kRowPoolCap) continue;
    const int64_t full = (ne + 63) / 64 * 64;
    const auto width = [&](int E, int64_t le) {
      return std::min(full, (row_need(E, excl, ne, le) + 63) / 64 * 64);
    };
    std::vector<std::vector<int32_t>> gs;
    std::vector<int64_t> w(Es.size(), 64);
    double gain = 0;
    for (size_t g0 = 0; g0 < v.size(); g0 += kWalkLibs) {
      std::vector<int32_t> grp;
      double save = 0;
      for (size_t k = g0; k < std::min(v.size(), g0 + kWalkLibs); ++k) {
        const Realization& R = p.rz[v[k]];
        if (width(Es.back(), R.l_eff) > kRowMaxW) continue;
        save += scan_cost(Emax, R.l_eff);
        for (int E : Es) save += scan_cost(E, 0);
        grp.push_back(v[k]);
      }
      if (grp.empty()) break;
      const int64_t le = p.rz[grp.back()].l_eff;
      for (int E : Es) save -= walk_cost(E, width(E, le) / 64);
      if (save <= 0) break;
      for (size_t e = 0; e < Es.size(); ++e) w[e] = std::max(w[e], width(Es[e], le));
      gain += save;
      gs.push_back(std::move(grp));
    }
    for (size_t e = 0; e < Es.size(); ++e) gain -= row_cost(Es[e], ne, w[e]);
    if (gs.empty() || gain <= 0) continue;
    gain_all += gain * (double)ne;
    n_groups += gs.size() * Es.size();
    groups.push_back(std::move(gs));
  }
  if (gain_all < kWalkMinGain || !groups_fit(p, n_groups)) return;

  for (auto& gs : groups)
    for (auto& grp : gs)
      for (int32_t r : grp) p.walked[r] = 1;
  la.sub_first = (int32_t)p.sub_launches.size();
  for (int E : Es) {
    std::vector<WalkPick> picks;
    for (auto& gs : groups) {
      WalkPick pk;
      for (auto& grp : gs) {
        const Realization& last = p.rz[grp.back()];
        const int64_t full = ((int64_t)last.n_e + 63) / 64 * 64;
        const int64_t w =
            std::min(full, (row_need(E, excl, last.n_e, last.l_eff) + 63) / 64 * 64);
        std::vector<int32_t> libs;
        for (int32_t r : grp) {
          Realization R = p.rz[r];
          R.E = E;
          R.tgt_off += (int64_t)(Emax - E) * R.tau;     // target at common point 0
          R.slot_base += (int64_t)(E - 1) * R.n_tiles;
          libs.push_back(add_walked(p, R, r));
        }
        pk.w = std::max(pk.w, w);
        pk.groups.push_back(std::move(libs));
        pk.chunks.push_back((int32_t)(w / 64));
      }
      picks.push_back(std::move(pk));
    }
    Launch sub{};
    sub.E = E;
    lay_out_walks(p, picks, sub, bits);
    p.sub_launches.push_back(sub);
  }
  la.sub_count = (int32_t)p.sub_launches.size() - la.sub_first;
}

// Waves, then the work items of each wave grouped by E (one launch each):
// the realizations that walk neighbour rows, and the scanned ones, the
// costliest first within a group: a scan costs n_query * l_eff pairs, a
// table walk about n_query * (E+1) n_e / l_eff row entries.
static void order_items(Plan& p) {
  split_waves(p);
  p.walked.assign(p.rz.size(), 0);
  p.want_table.resize(p.rz.size(), 0);
  if (p.spec.walk) p.walk_out.assign(p.rz.size(), WalkOut{});
  auto cost = [&](const Realization& R) {
    return R.table_off >= 0 ? (double)R.n_query * (R.E + 1) * R.n_e / R.l_eff / 8.0
                            : (double)R.n_query * R.l_eff;
  };
  for (size_t w = 0; w < p.waves.size(); ++w) {
    std::vector<int32_t> order(p.wave_rz.begin() + p.wave_rz_first[w],
                               p.wave_rz.begin() + p.wave_rz_first[w + 1]);
    std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) {
      if (p.rz[a].E != p.rz[b].E) return p.rz[a].E < p.rz[b].E;
      return cost(p.rz[a]) > cost(p.rz[b]);
    });
    p.waves[w].launch_first = (int32_t)p.launches.size();
    int64_t bits = 0;                 // words of the wave's bitmaps
    for (size_t a = 0; a < order.size();) {
      size_t b = a;
      while (b < order.size() && p.rz[order[b]].E == p.rz[order[a]].E) ++b;
      Launch la{};
      la.E = p.rz[order[a]].E;
      la.first = (int32_t)p.items.size();
      const std::vector<int32_t> group(order.begin() + a, order.begin() + b);
      if (p.shared_emax > 0)
        plan_shared_walks(p, group, la, bits);
      else
        plan_walks(p, group, la, bits);
      for (; a < b; ++a) {
        if (p.walked[order[a]] || (!p.nested.empty() && p.rz[order[a]].n_seg == 0)) continue;
        const Realization& R = p.rz[order[a]];
        for (int t = 0; t < R.n_tiles; ++t) p.items.push_back({order[a], t});
        la.count += R.n_tiles;
        if (p.items.size() > (size_t)INT32_MAX) fail(CCM_E_INVAL, "too many work items");
      }
      // few items: each lane's queries spread over more wavefronts
      int64_t l_max = 0;
      for (int32_t x = la.first; x < la.first + la.count; ++x)
        l_max = std::max<int64_t>(l_max, p.rz[p.items[x].rz].l_eff);
      const int q = crossmap_queries_per_lane(la.E);
      la.spread = p.spec.spread && p.spec.M == 0 && p.nested.empty() && p.shared_emax == 0 &&
                  p.tables.empty() && la.batch_count == 0 && la.count > 0 &&
                  la.count <= kSpreadItems &&
                  (double)l_max * (2 * la.E + 4) * (q - 1) >= kSpreadMinWork;
      if (la.spread)
        p.n_pred = std::max(p.n_pred,
                            (int64_t)la.count * kBlock * q);
      p.launches.push_back(la);
    }
    p.waves[w].launch_count = (int32_t)p.launches.size() - p.waves[w].launch_first;
    p.n_bits = std::max(p.n_bits, bits);
  }
  if (p.walk_groups.empty()) return;
  // a walked realization needs neither its draw as a list nor a gathered
  // library, but for library-point queries, whose order is the gathered one;
  // a chain needs the segments it still scans
  if (p.spec.query_set != 0) return;
  std::vector<char> skip(p.gather.size(), 0);
  if (!p.nested.empty()) {
    for (NestedJob& nj : p.nested) {
      if (nj.bits == 0) continue;
      nj.n_list = 0;
    }
    for (int32_t r : p.wave_rz) {
      const Realization& R = p.rz[r];
      NestedJob& nj = p.nested[p.rz_sample[r]];
      nj.n_list = std::max<int64_t>(nj.n_list, p.segs[R.seg_off + R.n_seg]);
      for (int k = R.n_seg; k < nj.n_seg; ++k) skip[p.rz_gather[r] + k] = 1;
    }
  } else {
    for (size_t r = 0; r < p.rz.size(); ++r)
      if (p.walked[r]) p.sample[p.rz_sample[r]].no_list = 1;
    for (size_t r = 0; r < p.rz.size(); ++r)
      if (!p.walked[r]) p.sample[p.rz_sample[r]].no_list = 0;
    for (size_t r = 0; r < p.rz.size(); ++r)
      if (p.walked[r]) skip[p.rz_gather[r]] = 1;
  }
  for (Wave& w : p.waves) {
    std::vector<GatherJob> keep;
    int64_t max_ne = 0;
    for (int64_t g = w.gather_first; g < w.gather_first + w.gather_count; ++g)
      if (!skip[g]) {
        keep.push_back(p.gather[g]);
        if (p.gather[g].sorted) max_ne = std::max(max_ne, p.gather[g].n_e);
      }
    std::copy(keep.begin(), keep.end(), p.gather.begin() + w.gather_first);
    w.gather_count = (int64_t)keep.size();
    w.max_sorted_n_e = max_ne;
  }
}

// Nested libraries: per (E, tau) the distinct library sizes, sorted, split
// one ordering per r into segments; per (r, direction) one chain whose
// segments are gathered separately (each in visiting order, with its own
// scan starts) and scanned in order, one snapshot per size.
static Plan make_plan_nested(const Spec& s) {
  if (s.query_set != 0) fail(CCM_E_INVAL, "nested libraries predict every embedded point");
  if (s.flags & (CCM_FLAG_TABLE | CCM_FLAG_PLAIN | CCM_FLAG_SHARED_E))
    fail(CCM_E_INVAL,
         "nested libraries do not combine with the table, plain or E-sweep-sharing forms");
  Plan p;
  p.spec = s;
  p.mode = excl_mode(s.excl);
  p.window = s.excl > 0 ? s.excl : 0;
  const int nE = (int)s.E.size(), nT = (int)s.tau.size(), nL = (int)s.L.size();
  const int64_t N = s.N;
  p.n64 = 2 * N;
  p.n32 = 2 * N;
  p.ingest.push_back({0, 0, 2 * N});
  const int64_t sorted_limit = gather_max_sorted_n_e();
  p.n_out = 2LL * nE * nT * nL * s.r;
  p.L_eff.assign((size_t)nE * nT * nL, 0);
  for (int ie = 0; ie < nE; ++ie) {
    const int32_t E = s.E[ie];
    const int Q = crossmap_queries_per_lane(E);
    const int64_t qt = (int64_t)kBlock * Q;
    for (int it = 0; it < nT; ++it) {
      const int32_t tau = s.tau[it];
      const int64_t ne = N - (int64_t)(E - 1) * tau;
      std::vector<int64_t> sizes;
      for (int il = 0; il < nL; ++il) {
        const int64_t le = std::min(s.L[il], ne);
        p.L_eff[((size_t)ie * nT + it) * nL + il] = le;
        sizes.push_back(le);
      }
      std::sort(sizes.begin(), sizes.end());
      sizes.erase(std::unique(sizes.begin(), sizes.end()), sizes.end());
      const int n_seg = (int)sizes.size();
      const int64_t lmax = sizes.back();
      const int64_t seg_off = (int64_t)p.segs.size();
      p.segs.push_back(0);
      for (int64_t z : sizes) p.segs.push_back((int32_t)z);
      int64_t emb_off[2], qord_off[2], ord_off[2];
      for (int sr = 0; sr < 2; ++sr) {
        emb_off[sr] = p.n_emb;
        qord_off[sr] = p.n_qord;
        ord_off[sr] = order_set(p, sr, embedding_order(E, tau));
        p.embed.push_back({sr * N, p.n_emb, ord_off[sr], p.n_qord, ne, N, E, tau, 0, 0});
        attach_kd(p, ord_off[sr], E, emb_off[sr], ne);
        p.n_emb += ne * E;
        p.n_qord += ne;
        p.max_embed = std::max(p.max_embed, ne * E);
      }
      const int32_t sorted = ne <= sorted_limit ? 1 : 0;
      if (sorted) p.max_sorted_n_e = std::max(p.max_sorted_n_e, ne);
      for (int ri = 0; ri < s.r; ++ri) {
        NestedJob nj{};
        nj.seed = s.seed;
        nj.n_e = ne;
        nj.n_out = lmax;
        nj.n_list = lmax;
        nj.seg_off = seg_off;
        nj.n_seg = n_seg;
        nj.out_off = p.n_lib;
        nj.scratch_off = p.n_scratch;
        nj.E = E;
        nj.tau = tau;
        nj.r_index = ri;
        p.nested.push_back(nj);
        p.n_lib += lmax;
        p.n_scratch += ne;
        for (int dir = 0; dir < 2; ++dir) {
          const int lib_s = dir == 0 ? 1 : 0;
          const int tgt_s = dir == 0 ? 0 : 1;
          Realization R{};
          R.emb_off = emb_off[lib_s];
          R.pts_off = p.n_pts;
          R.pj_off = p.n_pj;
          R.qord_off = qord_off[lib_s];
          R.tgt_off = tgt_s * N;
          R.E = E;
          R.tau = tau;
          R.n_e = (int32_t)ne;
          R.l_eff = (int32_t)lmax;
          R.n_query = (int32_t)ne;
          R.n_tiles = (int32_t)((ne + qt - 1) / qt);
          R.slot_base = p.n_slots;
          R.out_index = -1;
          R.table_off = -1;
          R.n_seg = n_seg;
          R.seg_off = seg_off;
          p.rz_sample.push_back((int64_t)p.nested.size() - 1);
          p.rz_gather.push_back((int64_t)p.gather.size());
          for (int k = 0; k < n_seg; ++k) {
            const int64_t b0 = p.segs[seg_off + k], b1 = p.segs[seg_off + k + 1];
            GatherJob gj{};
            gj.emb_off = R.emb_off;
            gj.lib_off = nj.out_off + b0;
            gj.order_off = ord_off[lib_s];
            gj.pts_off = R.pts_off + b0 * E;
            gj.pj_off = R.pj_off + b0;
            gj.start_off = (R.slot_base + (int64_t)k * R.n_tiles) * kWaves;
            gj.l_eff = b1 - b0;
            gj.n_e = ne;
            gj.n_series = N;
            gj.E = E;
            gj.tau = tau;
            gj.qt = (int32_t)qt;
            gj.query_set = 0;
            gj.sorted = sorted;
            p.gather.push_back(gj);
          }
          for (int il = 0; il < nL; ++il) {
            const int64_t le = p.L_eff[((size_t)ie * nT + it) * nL + il];
            const int k = (int)(std::lower_bound(sizes.begin(), sizes.end(), le) - sizes.begin());
            Realization F{};
            F.slot_base = R.slot_base + (int64_t)k * R.n_tiles;
            F.n_tiles = R.n_tiles;
            F.out_index = ((((int64_t)dir * nE + ie) * nT + it) * nL + il) * s.r + ri;
            p.rz_fin.push_back(F);
            p.preds += (double)ne;
          }
          p.n_pts += lmax * E;
          p.n_pj += lmax;
          p.n_slots += (int64_t)R.n_tiles * n_seg;
          p.rz.push_back(R);
          double pairs = (double)ne * (double)lmax;
          if (p.mode == kExclSelf) pairs -= (double)lmax;
          p.pairs += pairs;
          p.flops += pairs * (3.0 * E - 1.0);
        }
      }
    }
  }
  p.n_rho = (int64_t)p.rz_fin.size();
  if (p.rz.size() > (size_t)INT32_MAX) fail(CCM_E_INVAL, "too many realizations");
  order_items(p);
  p.device_bytes = p.n64 * 8 + p.n32 * 4 + p.n_emb * 4 + p.n_lib * 4 + p.n_pts * 4 + p.n_pred * 8 +
                   p.n_pj * 4 + p.n_qord * 4 + p.n_slots * 4 * kWaves +
                   (size_t)p.n_ord * 16 + p.n_scratch * 4 + p.segs.size() * 4 +
                   p.n_slots * sizeof(Moments) + p.n_out * 8 +
                   (p.rz.size() + p.rz_fin.size()) * sizeof(Realization) +
                   p.items.size() * sizeof(Item) + p.nested.size() * sizeof(NestedJob) +
                   p.gather.size() * sizeof(GatherJob) + p.walk_bytes();
  return p;
}

// E-sweep sharing: per tau, the embedding of E_max (the largest E asked for)
// over N_c points, one library per (L, r) drawn over them, and one
// realization per (L, r, direction) whose scan keeps a running list for
// every E <= E_max (moments slots: E_max per tile, E's at slot_base +
// (E-1) n_tiles); rz_fin holds one record per requested (E, L, r, direction).
static Plan make_plan_shared(const Spec& s) {
  if (s.query_set != 0) fail(CCM_E_INVAL, "E-sweep sharing predicts every embedded point");
  if (s.flags & (CCM_FLAG_TABLE | CCM_FLAG_PLAIN | CCM_FLAG_NESTED))
    fail(CCM_E_INVAL, "E-sweep sharing does not combine with the table, nested or plain forms");
  Plan p;
  p.spec = s;
  p.mode = excl_mode(s.excl);
  p.window = s.excl > 0 ? s.excl : 0;
  const int nE = (int)s.E.size(), nT = (int)s.tau.size(), nL = (int)s.L.size();
  const int64_t N = s.N;
  const int32_t Emax = *std::max_element(s.E.begin(), s.E.end());
  p.shared_emax = Emax;
  p.n64 = 2 * N;
  p.n32 = 2 * N;
  p.ingest.push_back({0, 0, 2 * N});
  const int64_t sorted_limit = gather_max_sorted_n_e();
  p.n_out = 2LL * nE * nT * nL * s.r;
  p.L_eff.assign((size_t)nE * nT * nL, 0);
  const int64_t qt = (int64_t)kBlock * shared_queries_per_lane(Emax);
  for (int it = 0; it < nT; ++it) {
    const int32_t tau = s.tau[it];
    const int64_t nc = N - (int64_t)(Emax - 1) * tau;
    int64_t emb_off[2], qord_off[2], ord_off[2];
    for (int sr = 0; sr < 2; ++sr) {
      emb_off[sr] = p.n_emb;
      qord_off[sr] = p.n_qord;
      ord_off[sr] = order_set(p, sr, shared_order(Emax, tau));
      p.embed.push_back({sr * N, p.n_emb, ord_off[sr], p.n_qord, nc, N, Emax, tau, 0, 0});
      p.n_emb += nc * Emax;
      p.n_qord += nc;
      p.max_embed = std::max(p.max_embed, nc * Emax);
    }
    const int32_t sorted = nc <= sorted_limit ? 1 : 0;
    if (sorted) p.max_sorted_n_e = std::max(p.max_sorted_n_e, nc);
    for (int il = 0; il < nL; ++il) {
      const int64_t le = std::min(s.L[il], nc);
      for (int ie = 0; ie < nE; ++ie) p.L_eff[((size_t)ie * nT + it) * nL + il] = le;
      for (int ri = 0; ri < s.r; ++ri) {
        const int64_t lib_off = p.n_lib;
        p.sample.push_back({s.seed, lib_off, 0, (int32_t)nc, (int32_t)le, 0, tau, ri, 0});
        p.n_lib += le;
        for (int dir = 0; dir < 2; ++dir) {
          const int lib_s = dir == 0 ? 1 : 0;
          const int tgt_s = dir == 0 ? 0 : 1;
          Realization R{};
          R.emb_off = emb_off[lib_s];
          R.pts_off = p.n_pts;
          R.pj_off = p.n_pj;
          R.qord_off = qord_off[lib_s];
          R.tgt_off = tgt_s * N;
          R.E = Emax;
          R.tau = tau;
          R.n_e = (int32_t)nc;
          R.l_eff = (int32_t)le;
          R.n_query = (int32_t)nc;
          R.n_tiles = (int32_t)((nc + qt - 1) / qt);
          R.slot_base = p.n_slots;
          R.out_index = -1;
          R.table_off = -1;
          GatherJob gj{};
          gj.emb_off = R.emb_off;
          gj.lib_off = lib_off;
          gj.order_off = ord_off[lib_s];
          gj.pts_off = R.pts_off;
          gj.pj_off = R.pj_off;
          gj.start_off = R.slot_base * kWaves;
          gj.l_eff = le;
          gj.n_e = nc;
          gj.n_series = N;
          gj.E = Emax;
          gj.tau = tau;
          gj.qt = (int32_t)qt;
          gj.query_set = 0;
          gj.sorted = sorted;
          p.gather.push_back(gj);
          for (int ie = 0; ie < nE; ++ie) {
            Realization F{};
            F.slot_base = R.slot_base + (int64_t)(s.E[ie] - 1) * R.n_tiles;
            F.n_tiles = R.n_tiles;
            F.out_index = ((((int64_t)dir * nE + ie) * nT + it) * nL + il) * s.r + ri;
            p.rz_fin.push_back(F);
            p.preds += (double)nc;
          }
          p.n_pts += le * Emax;
          p.n_pj += le;
          p.n_slots += (int64_t)R.n_tiles * Emax;
          p.rz.push_back(R);
          p.rz_sample.push_back((int64_t)p.sample.size() - 1);
          p.rz_gather.push_back((int64_t)p.gather.size() - 1);
          // each pair's E_max-coordinate distance is computed once
          double pairs = (double)nc * (double)le;
          if (p.mode == kExclSelf) pairs -= (double)le;
          p.pairs += pairs;
          p.flops += pairs * (3.0 * Emax - 1.0);
        }
      }
    }
  }
  p.n_rho = (int64_t)p.rz_fin.size();
  if (p.rz.size() > (size_t)INT32_MAX) fail(CCM_E_INVAL, "too many realizations");
  order_items(p);
  p.device_bytes = p.n64 * 8 + p.n32 * 4 + p.n_emb * 4 + p.n_lib * 4 + p.n_pts * 4 + p.n_pred * 8 +
                   p.n_pj * 4 + p.n_qord * 4 + p.n_slots * 4 * kWaves +
                   (size_t)p.n_ord * 16 + p.n_slots * sizeof(Moments) + p.n_out * 8 +
                   (p.rz.size() + p.rz_fin.size()) * sizeof(Realization) +
                   p.items.size() * sizeof(Item) + p.sample.size() * sizeof(SampleJob) +
                   p.gather.size() * sizeof(GatherJob) + p.walk_bytes();
  return p;
}

// Validate a sweep and lay out every realization of it.
Plan make_plan(const Spec& s) {
  if (s.N < 2) fail(CCM_E_INVAL, "N must be >= 2");
  if (s.E.empty() || s.tau.empty() || s.L.empty()) fail(CCM_E_INVAL, "empty E, tau or L list");
  if (s.r < 1) fail(CCM_E_INVAL, "r must be >= 1");
  if (s.query_set != 0 && s.query_set != 1) fail(CCM_E_INVAL, "query_set must be 0 or 1");
  if (s.N > (int64_t)INT32_MAX / 2) fail(CCM_E_INVAL, "N too large");
  for (int32_t e : s.E)
    if (e < 1 || e > kMaxE) fail(CCM_E_INVAL, "E must be in [1, 10]");
  for (int32_t t : s.tau)
    if (t < 1) fail(CCM_E_INVAL, "tau must be >= 1");
  for (int32_t e : s.E)
    for (int32_t t : s.tau) {
      const int64_t ne = s.N - (int64_t)(e - 1) * t;
      if (ne < e + 2) fail(CCM_E_INVAL, "N_e = N - (E-1) tau must be >= E + 2");
      for (int64_t l : s.L) {
        if (l < e + 2) fail(CCM_E_INVAL, "every L must be >= E + 2");
        if (std::min(l, ne) < min_library(e, s.excl))
          fail(CCM_E_INVAL, "library too small for the exclusion window");
      }
    }
  if (s.flags & CCM_FLAG_NESTED) return make_plan_nested(s);
  if (s.flags & CCM_FLAG_SHARED_E) return make_plan_shared(s);

  Plan p;
  p.spec = s;
  p.mode = excl_mode(s.excl);
  p.window = s.excl > 0 ? s.excl : 0;
  const int nE = (int)s.E.size(), nT = (int)s.tau.size(), nL = (int)s.L.size();
  const int64_t N = s.N;
  p.n64 = 2 * N;
  p.n32 = 2 * N;
  p.ingest.push_back({0, 0, 2 * N});
  const int64_t sorted_limit = gather_max_sorted_n_e();
  p.n_out = 2LL * nE * nT * nL * s.r;
  p.L_eff.assign((size_t)nE * nT * nL, 0);

  for (int ie = 0; ie < nE; ++ie) {
    const int32_t E = s.E[ie];
    const int Q = crossmap_queries_per_lane(E);
    const int64_t qt = (int64_t)kBlock * Q;
    for (int it = 0; it < nT; ++it) {
      const int32_t tau = s.tau[it];
      const int64_t ne = N - (int64_t)(E - 1) * tau;
      int64_t emb_off[2], qord_off[2], ord_off[2];
      for (int sr = 0; sr < 2; ++sr) {
        emb_off[sr] = p.n_emb;
        qord_off[sr] = p.n_qord;
        ord_off[sr] = order_set(p, sr, embedding_order(E, tau));
        p.embed.push_back({sr * N, p.n_emb, ord_off[sr], p.n_qord, ne, N, E, tau, 0, 0});
        attach_kd(p, ord_off[sr], E, emb_off[sr], ne);
        p.n_emb += ne * E;
        p.n_qord += ne;
        p.max_embed = std::max(p.max_embed, ne * E);
      }
      const int32_t sorted = ne <= sorted_limit ? 1 : 0;
      if (sorted) p.max_sorted_n_e = std::max(p.max_sorted_n_e, ne);
      for (int il = 0; il < nL; ++il) {
        const int64_t le = std::min(s.L[il], ne);
        p.L_eff[((size_t)ie * nT + it) * nL + il] = le;
        for (int ri = 0; ri < s.r; ++ri) {
          const int64_t lib_off = p.n_lib;
          p.sample.push_back({s.seed, lib_off, 0, (int32_t)ne, (int32_t)le, E, tau, ri, 0});
          p.n_lib += le;
          for (int dir = 0; dir < 2; ++dir) {
            // dir 0: library Y (series 1) predicts X (series 0); dir 1: reverse
            const int lib_s = dir == 0 ? 1 : 0;
            const int tgt_s = dir == 0 ? 0 : 1;
            Realization R{};
            R.emb_off = emb_off[lib_s];
            R.pts_off = p.n_pts;
            R.pj_off = p.n_pj;
            R.qord_off = qord_off[lib_s];
            R.tgt_off = tgt_s * N;
            R.E = E;
            R.tau = tau;
            R.n_e = (int32_t)ne;
            R.l_eff = (int32_t)le;
            R.n_query = (int32_t)(s.query_set ? le : ne);
            R.n_tiles = (int32_t)((R.n_query + qt - 1) / qt);
            R.slot_base = p.n_slots;
            R.out_index = ((((int64_t)dir * nE + ie) * nT + it) * nL + il) * s.r + ri;
            R.table_off = -1;
            const bool table = use_table(p, E, ne, le);
            p.want_table.push_back(table && s.walk);
            if (table && !s.walk) {
              R.table_off = table_for(p, R.emb_off, ne, E);
              R.table_w = (int32_t)std::min<int64_t>(kTableWidth, ne);
              p.e_table_ne[E] = std::max(p.e_table_ne[E], (int)ne);
              p.table_rz += 1;
            }
            GatherJob gj{};
            gj.emb_off = R.emb_off;
            gj.lib_off = lib_off;
            gj.order_off = ord_off[lib_s];
            gj.pts_off = R.pts_off;
            gj.pj_off = R.pj_off;
            gj.start_off = R.slot_base * kWaves;
            gj.l_eff = le;
            gj.n_e = ne;
            gj.n_series = N;
            gj.E = E;
            gj.tau = tau;
            gj.qt = (int32_t)qt;
            gj.query_set = s.query_set;
            gj.sorted = sorted;
            p.gather.push_back(gj);
            p.n_pts += le * E;
            p.n_pj += le;
            p.n_slots += R.n_tiles;
            p.rz.push_back(R);
            p.rz_sample.push_back((int64_t)p.sample.size() - 1);
            p.rz_gather.push_back((int64_t)p.gather.size() - 1);
            // algorithmic work: every (query, candidate) pair but the query itself
            const double nq = (double)R.n_query;
            double pairs = nq * (double)le;
            if (p.mode == kExclSelf) pairs -= s.query_set ? nq : (double)le;
            p.pairs += pairs;
            p.flops += pairs * (3.0 * E - 1.0);
            p.preds += nq;
          }
        }
      }
    }
  }
  if (p.rz.size() > (size_t)INT32_MAX) fail(CCM_E_INVAL, "too many realizations");
  p.n_rho = (int64_t)p.rz.size();

  order_items(p);

  p.device_bytes = p.n64 * 8 + p.n32 * 4 + p.n_emb * 4 + p.n_lib * 4 + p.n_pts * 4 + p.n_pred * 8 +
                   p.n_pj * 4 + p.n_qord * 4 + p.n_slots * 4 * kWaves +
                   (size_t)p.n_ord * 16 + p.n_table * 4 + p.tables.size() * sizeof(TableJob) +
                   p.n_slots * sizeof(Moments) + p.n_out * 8 +
                   p.rz.size() * sizeof(Realization) + p.items.size() * sizeof(Item) +
                   p.sample.size() * sizeof(SampleJob) + p.gather.size() * sizeof(GatherJob) +
                   p.walk_bytes();
  return p;
}

// Causal matrix: M series, one (E, tau); libraries per (L, r) shared by every
// series; one realization per (searched series, L, r) predicting all others.
Plan make_plan_matrix(const Spec& s) {
  if (s.M < 2) fail(CCM_E_INVAL, "M must be >= 2");
  if (s.flags & (CCM_FLAG_NESTED | CCM_FLAG_SHARED_E))
    fail(CCM_E_INVAL, "nested libraries and E-sweep sharing are not supported by the matrix form");
  if (s.N < 2) fail(CCM_E_INVAL, "N must be >= 2");
  if (s.L.empty()) fail(CCM_E_INVAL, "empty L list");
  if (s.r < 1) fail(CCM_E_INVAL, "r must be >= 1");
  if (s.query_set != 0 && s.query_set != 1) fail(CCM_E_INVAL, "query_set must be 0 or 1");
  // the kernel addresses the time-major target table (N rows of
  // target_stride(M) doubles) with 32-bit byte offsets
  if ((int64_t)target_stride(s.M) * s.N > ((int64_t)1 << 29))
    fail(CCM_E_INVAL, "M*N too large (the target table must stay within 4 GiB)");
  const int32_t E = s.E[0], tau = s.tau[0];
  if (E < 1 || E > kMaxE) fail(CCM_E_INVAL, "E must be in [1, 10]");
  if (tau < 1) fail(CCM_E_INVAL, "tau must be >= 1");
  const int64_t N = s.N;
  const int64_t ne = N - (int64_t)(E - 1) * tau;
  if (ne < E + 2) fail(CCM_E_INVAL, "N_e = N - (E-1) tau must be >= E + 2");
  for (int64_t l : s.L) {
    if (l < E + 2) fail(CCM_E_INVAL, "every L must be >= E + 2");
    if (std::min(l, ne) < min_library(E, s.excl))
      fail(CCM_E_INVAL, "library too small for the exclusion window");
  }
  Plan p;
  p.spec = s;
  p.mode = excl_mode(s.excl);
  p.window = s.excl > 0 ? s.excl : 0;
  const int M = s.M, nL = (int)s.L.size();
  p.n64 = (int64_t)M * N;
  p.n32 = (int64_t)M * N;
  p.ingest.push_back({0, 0, (int64_t)M * N});
  p.n_out = (int64_t)M * M * nL * s.r;
  p.L_eff.assign(nL, 0);
  const int Q = crossmap_queries_per_lane(E);
  const int64_t qt = (int64_t)kBlock * Q;
  const int32_t sorted = ne <= gather_max_sorted_n_e() ? 1 : 0;
  if (sorted) p.max_sorted_n_e = ne;
  std::vector<int64_t> emb_off(M), qord_off(M), ord_off(M);
  for (int a = 0; a < M; ++a) {
    emb_off[a] = p.n_emb;
    qord_off[a] = p.n_qord;
    ord_off[a] = order_set(p, a, embedding_order(E, tau));
    p.embed.push_back({a * N, p.n_emb, ord_off[a], p.n_qord, ne, N, E, tau, 0, 0});
    attach_kd(p, ord_off[a], E, emb_off[a], ne);
    p.n_emb += ne * E;
    p.n_qord += ne;
    p.max_embed = std::max(p.max_embed, ne * E);
  }
  std::vector<int64_t> lib_off((size_t)nL * s.r);
  for (int il = 0; il < nL; ++il) {
    const int64_t le = std::min(s.L[il], ne);
    p.L_eff[il] = le;
    for (int ri = 0; ri < s.r; ++ri) {
      lib_off[(size_t)il * s.r + ri] = p.n_lib;
      p.sample.push_back({s.seed, p.n_lib, 0, (int32_t)ne, (int32_t)le, E, tau, ri, 0});
      p.n_lib += le;
    }
  }
  for (int a = 0; a < M; ++a)
    for (int il = 0; il < nL; ++il)
      for (int ri = 0; ri < s.r; ++ri) {
        const int64_t le = p.L_eff[il];
        Realization R{};
        R.emb_off = emb_off[a];
        R.pts_off = p.n_pts;
        R.pj_off = p.n_pj;
        R.qord_off = qord_off[a];
        R.tgt_off = 0;
        R.E = E;
        R.tau = tau;
        R.n_e = (int32_t)ne;
        R.l_eff = (int32_t)le;
        R.n_query = (int32_t)(s.query_set ? le : ne);
        R.n_tiles = (int32_t)((R.n_query + qt - 1) / qt);
        R.slot_base = p.n_slots;
        R.out_index = (((int64_t)a * M) * nL + il) * s.r + ri;   // target 0 of row a
        R.table_off = -1;
        const bool table = use_table(p, E, ne, le);
        p.want_table.push_back(table && s.walk);
        if (table && !s.walk) {
          R.table_off = table_for(p, R.emb_off, ne, E);
          R.table_w = (int32_t)std::min<int64_t>(kTableWidth, ne);
          p.e_table_ne[E] = std::max(p.e_table_ne[E], (int)ne);
          p.table_rz += M - 1;   // rho values, like n_rho
        }
        GatherJob gj{};
        gj.emb_off = R.emb_off;
        gj.lib_off = lib_off[(size_t)il * s.r + ri];
        gj.order_off = ord_off[a];
        gj.pts_off = R.pts_off;
        gj.pj_off = R.pj_off;
        gj.start_off = R.slot_base * kWaves;
        gj.l_eff = le;
        gj.n_e = ne;
        gj.n_series = N;
        gj.E = E;
        gj.tau = tau;
        gj.qt = (int32_t)qt;
        gj.query_set = s.query_set;
        gj.sorted = sorted;
        p.gather.push_back(gj);
        p.n_pts += le * E;
        p.n_pj += le;
        p.n_slots += R.n_tiles;
        p.rz.push_back(R);
        p.self_of.push_back(a);
        p.rz_sample.push_back((int64_t)il * s.r + ri);
        p.rz_gather.push_back((int64_t)p.gather.size() - 1);
        const double nq = (double)R.n_query;
        double pairs = nq * (double)le;
        if (p.mode == kExclSelf) pairs -= s.query_set ? nq : (double)le;
        p.pairs += pairs;
        p.flops += pairs * (3.0 * E - 1.0);
        p.preds += nq * (M - 1);
      }
  p.n_rho = (int64_t)p.rz.size() * (M - 1);
  order_items(p);
  p.device_bytes = p.n64 * 8 + p.n32 * 4 + p.n_ord * 16 + p.n_emb * 4 + p.n_lib * 4 +
                   p.n_pts * 4 + p.n_pred * 8 +
                   p.n_pj * 4 + p.n_qord * 4 + p.n_slots * 4 * kWaves +
                   p.n_slots * M * multi_sums_bytes() + p.n_out * 8 +
                   N * target_stride(M) * 8 + p.n_table * 4 +
                   p.tables.size() * sizeof(TableJob) +
                   p.rz.size() * (sizeof(Realization) + 4) + p.items.size() * sizeof(Item) +
                   p.sample.size() * sizeof(SampleJob) + p.gather.size() * sizeof(GatherJob) +
                   p.walk_bytes();
  return p;
}

void check_host_series(const double* s, int64_t n, const char* name) {
  if (!s) fail(CCM_E_INVAL, std::string(name) + " is NULL");
  for (int64_t t = 0; t < n; ++t)
    if (!std::isfinite(s[t]) || std::fabs(s[t]) > 1e17)
      fail(CCM_E_INVAL, std::string(name) + " has a non-finite or too large value");
}

Spec make_spec(int64_t N, const int32_t* E, int32_t nE, const int32_t* tau, int32_t ntau,
               const int64_t* L, int32_t nL, int32_t r, uint64_t seed,
               const ccm_opts* opts) {
  if (!E || !tau || !L) fail(CCM_E_INVAL, "NULL parameter array");
  if (nE < 1 || ntau < 1 || nL < 1) fail(CCM_E_INVAL, "nE, ntau and nL must be >= 1");
  Spec s;
  s.N = N;
  s.E.assign(E, E + nE);
  s.tau.assign(tau, tau + ntau);
  s.L.assign(L, L + nL);
  s.r = r;
  s.seed = seed;
  if (opts) {
    s.excl = opts->exclusion_radius;
    s.query_set = opts->query_set;
    s.flags = opts->flags;
  }
  return s;
}


}  // namespace ccmh
