// ccm_walk.h -- device templates of the neighbour-row path: the sorted
// neighbour rows of an embedding, the walk of a row by 64 libraries at once,
// and the moments of the predictions it leaves (one translation unit per
// embedding dimension instantiates them, see ccm_inst_walk.hip).
//
// A query's neighbours in any library are the first E+1 members of that
// library (not excluded) in the query's row: every embedded point in (d2, j)
// order.  The rows do not depend on the library, so a call with many
// libraries per embedding (L list times r) pays for the search once per
// query instead of once per query and library; what is left per library is
// a walk of about (E+1) n_e / l_eff row entries.  The rows hold the same
// binary32 d2 as the scan and the order is the same total order, so the
// neighbours, and with the same operations in the same order the
// predictions, moments and rho, are the scan's bit for bit.
#pragma once
#include "ccm_device.h"

namespace ccmk {

// ---------------------------------------------------------------------------
// neighbour rows
// ---------------------------------------------------------------------------

// The points of one embedding in visiting order, one array per coordinate
// (float [E][n_e]), and the bounding box of every run of 64 of them (float
// [E] lowest, then [E] highest, at box_slot(run)).  One wavefront per run.
// Run 4 l + v of every 256 is looked at by lane l of wavefront v of the row
// kernel: its box lies where the wavefront reads consecutive ones.  (One
// array per coordinate instead: 3.5 against 2.1 ms for 2 x 10^5 rows at E = 3.)
__device__ __forceinline__ int box_slot(int run) {
  return (run & ~255) + ((run & 3) << 6) + ((run & 255) >> 2);
}

template <int E>
__global__ __launch_bounds__(kBlock) void k_order_points(const RowJob* __restrict__ jobs,
                                                         const float* __restrict__ emb_pool,
                                                         const int32_t* __restrict__ qord_pool,
                                                         float* __restrict__ pts_pool,
                                                         float* __restrict__ box_pool,
                                                         int* __restrict__ todo_n) {
  const RowJob J = jobs[blockIdx.y];
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *todo_n = 0;   // for k_rows
  const int lane = threadIdx.x & 63;
  const int b = blockIdx.x * kWaves + (threadIdx.x >> 6);
  if (b * 64 >= J.n_e) return;
  const int p = min(b * 64 + lane, J.n_e - 1);     // the tail repeats the last point
  const int i = qord_pool[J.qord_off + p];
  const float* __restrict__ v = emb_pool + J.emb_off + (int64_t)i * J.stride;
  float* __restrict__ o = pts_pool + J.pts_off;
  float* __restrict__ box = box_pool + J.box_off + (int64_t)box_slot(b) * (2 * E);
#pragma unroll
  for (int k = 0; k < E; ++k) {
    const float x = v[k];
    o[(int64_t)k * J.n_e + p] = x;
    float lo = x, hi = x;
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) {
      lo = fminf(lo, __shfl_xor(lo, s, 64));
      hi = fmaxf(hi, __shfl_xor(hi, s, 64));
    }
    if (lane == 0) {
      box[k] = lo;
      box[E + k] = hi;
    }
  }
}

// LDS of the row kernel (dynamic): four candidate segments of seg keys, one
// per wavefront, in which the keys are later grouped by bucket; bucket
// counters.  Room for 2 w + 768 keys, at most eleven per thread.
constexpr int kRowBuckets = 1024;
constexpr uint32_t kRowCrowd = 96;               // larger buckets: by octave instead
constexpr uint32_t kRowMost = 384;               // largest bucket ordered by comparison
constexpr float kRowTarget = 1.5f;               // candidates aimed at, times w
constexpr int kRowPerThread = 11;
constexpr int row_segment(int w) { return w / 2 + 192; }
static_assert(kWaves * row_segment(kRowMaxW) <= kRowPerThread * kBlock, "keys held in registers");
inline size_t row_lds_bytes(int w) {
  return (size_t)kWaves * row_segment(w) * 8 + kRowBuckets * 4;
}

// Distances of the lanes' points of run b to the query.
template <int E>
__device__ __forceinline__ float run_d2(const float* __restrict__ pts, int n_e, int c,
                                        const float (&q)[E]) {
  float d = q[0] - pts[c];
  float acc = d * d;
#pragma unroll
  for (int k = 1; k < E; ++k) {
    d = q[k] - pts[(int64_t)k * n_e + c];
    acc = __builtin_fmaf(d, d, acc);
  }
  return acc;
}

// A lower bound of run b's distances: the same binary32 chain over the gap
// between the query and the run's box.  Subtraction, product and fused
// multiply-add round monotonically, so no point of the box has a smaller d2.
template <int E>
__device__ __forceinline__ float run_bound(const float* __restrict__ box, const float (&q)[E]) {
  float acc = 0.f;
#pragma unroll
  for (int k = 0; k < E; ++k) {
    const float g = fmaxf(fmaxf(box[k] - q[k], q[k] - box[E + k]), 0.f);
    acc = k == 0 ? g * g : __builtin_fmaf(g, g, acc);
  }
  return acc;
}

__device__ __forceinline__ uint64_t row_key(float d2, int j) {
  return ((uint64_t)__float_as_uint(d2) << 32) | (uint32_t)j;
}
// Bucket of a key: by d2 scaled to the threshold, or (scale < 0) by its binary
// exponent and leading mantissa bits, 32 to the octave below the threshold.
__device__ __forceinline__ int row_bucket(uint64_t key, float scale, uint32_t base) {
  const uint32_t u = (uint32_t)(key >> 32);
  if (scale < 0.f) return u <= base ? 0 : min(kRowBuckets - 1, (int)((u - base) >> 18));
  const float x = __uint_as_float(u) * scale;
  return x < (float)(kRowBuckets - 1) ? (int)x : (x >= 0.f ? kRowBuckets - 1 : 0);
}

// Calls f(c, d2, valid) for the 64 points c of every run whose bound does
// not exceed t, runs dealt to the workgroup's wavefronts in turn.  Four runs
// are loaded together: one at a time, the wavefronts waited on their loads
// for most of the pass (2 x 5 x 10^4 rows of 10^4 points at E = 10: 4.5
// against 3.2 ms).
template <int E, class F>
__device__ __forceinline__ void visit_runs(const float* __restrict__ pts,
                                           const float* __restrict__ boxes, int n_e,
                                           const float (&q)[E], float t, F&& f) {
  constexpr int kTogether = 4;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nb = (n_e + 63) >> 6;
  int run[kTogether];                              // found and not yet visited
#pragma unroll
  for (int u = 0; u < kTogether; ++u) run[u] = 0;
  int found = 0;
  const auto visit = [&] {
    float d2[kTogether];
#pragma unroll
    for (int u = 0; u < kTogether; ++u)
      d2[u] = run_d2<E>(pts, n_e, min(run[u] * 64 + lane, n_e - 1), q);
#pragma unroll
    for (int u = 0; u < kTogether; ++u)
      if (u < found) f(run[u] * 64 + lane, d2[u], run[u] * 64 + lane < n_e);
    found = 0;
  };
  for (int g = 0; g < nb; g += kBlock) {
    const int b = g + lane * kWaves + wave;
    // (slots past the last run are read and ignored)
    const bool near =
        run_bound<E>(boxes + (int64_t)(g + wave * 64 + lane) * (2 * E), q) <= t && b < nb;
    uint64_t open = __builtin_amdgcn_ballot_w64(near);
    while (open) {
      const int r = g + __builtin_ctzll(open) * kWaves + wave;
      open &= open - 1ull;
#pragma unroll
      for (int u = 0; u < kTogether; ++u)
        if (u == found) run[u] = r;
      if (++found == kTogether) visit();
    }
  }
  if (found) visit();
}

// The farthest of the w points around position p in visiting order: a bound of
// its w-th distance, infinite with a NaN among them (the whole workgroup; two
// barriers, s_n is used).
template <int E>
__device__ __forceinline__ float order_reach(const float* __restrict__ pts, int n, int w, int p,
                                             const float (&q)[E], int* s_n) {
  const int tid = threadIdx.x;
  const int a = max(0, min(p - w / 2, n - w));
  uint32_t bits = 0u;                              // (a NaN's lie above infinity's)
  for (int c = a + tid; c < a + w; c += kBlock)
    bits = max(bits, __float_as_uint(run_d2<E>(pts, n, c, q)) & 0x7fffffffu);
  float m = __uint_as_float(min(bits, 0x7f800000u));
#pragma unroll
  for (int s = 32; s > 0; s >>= 1) m = fmaxf(m, __shfl_xor(m, s, 64));
  __syncthreads();
  if ((tid & 63) == 0) s_n[tid >> 6] = __float_as_int(m);
  __syncthreads();
  m = 0.f;
#pragma unroll
  for (int v = 0; v < kWaves; ++v) m = fmaxf(m, __int_as_float(s_n[v]));
  return m;
}

// Rows among repeated values, where many points share a distance: the
// distances in ascending order from 0 (the query's own), one pass over the
// runs within reach (at least the w-th distance) for each, which marks the
// points at this distance in a bitmap over their indices and finds the next
// one; the marked indices are the row's next entries, in order.  Given up
// (false) when the distances bring fewer than w / 16 points each.  The bitmap
// takes `words` 32-bit words of LDS; longer series take more passes per
// distance.  The whole workgroup.
template <int E>
__device__ bool row_by_level(const float* __restrict__ pts, const float* __restrict__ boxes,
                             const int32_t* __restrict__ qord, int n, int w, const float (&q)[E],
                             float reach, uint32_t* bits, int words,
                             uint64_t* __restrict__ row) {
  __shared__ uint32_t s_min;
  __shared__ int s_cnt[kWaves];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t far = __float_as_uint(__builtin_inff());
  int filled = 0;
  uint32_t T = 0u;                                 // bits of this distance
  for (int level = 0;; ++level) {
    if (tid == 0) s_min = far;
    uint32_t next = far;
    for (int j0 = 0; j0 < n; j0 += words * 32) {
      const int nw = min(words, (n - j0 + 31) >> 5);
      for (int x = tid; x < nw; x += kBlock) bits[x] = 0u;
      __syncthreads();
      visit_runs<E>(pts, boxes, n, q, reach, [&](int c, float d2, bool valid) {
        if (!valid) return;
        const uint32_t u = __float_as_uint(d2);
        if (u > T) {
          next = min(next, u);
        } else if (u == T) {
          const int j = qord[c] - j0;
          if (j >= 0 && j < nw * 32) atomicOr(&bits[j >> 5], 1u << (j & 31));
        }
      });
      __syncthreads();
      // the marked indices, consecutive words per thread
      const int per = (nw + kBlock - 1) / kBlock;
      int sum = 0;
      for (int x = tid * per; x < min((tid + 1) * per, nw); ++x) sum += __popc(bits[x]);
      int inc = sum;
#pragma unroll
      for (int s = 1; s < 64; s <<= 1) {
        const int y = __shfl_up(inc, s, 64);
        if (lane >= s) inc += y;
      }
      if (lane == 63) s_cnt[wave] = inc;
      __syncthreads();
      int at = filled + inc - sum, all = 0;
#pragma unroll
      for (int v = 0; v < kWaves; ++v) {
        if (v < wave) at += s_cnt[v];
        all += s_cnt[v];
      }
      for (int x = tid * per; x < min((tid + 1) * per, nw) && at < w; ++x) {
        uint32_t b = bits[x];
        while (b && at < w) {
          row[at++] = ((uint64_t)T << 32) | (uint32_t)(j0 + x * 32 + __builtin_ctz(b));
          b &= b - 1u;
        }
      }
      filled += all;
      __syncthreads();
      if (filled >= w) return true;
    }
    if (filled * 16 < (level + 1) * w) return false;
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) next = min(next, (uint32_t)__shfl_xor((int)next, s, 64));
    if (lane == 0) atomicMin(&s_min, next);
    __syncthreads();
    T = s_min;
    __syncthreads();
    if (T == far) return false;                    // (reach below the w-th distance)
  }
}

// Rows with no end to their distances among the repeated ones: radix select of
// the w-th distance (four 8-bit passes over the runs that can hold it), then
// the nearer points and the lowest-index ones at it, sorted in `grouped`
// (room for the power of two >= w).  hist: 256 counters.  The whole
// workgroup.
template <int E>
__device__ void row_by_select(const float* __restrict__ pts, const float* __restrict__ boxes,
                               const int32_t* __restrict__ qord, int n, int w,
                               const float (&q)[E], float reach, uint64_t* grouped,
                               uint32_t* hist, uint64_t* __restrict__ row) {
  __shared__ uint32_t s_pick[3];
  __shared__ int s_at;
  const int tid = threadIdx.x;
  uint32_t prefix = 0u, mask = 0u, need = (uint32_t)w, at_T = 0u;
  // the counter that holds the need-th entry, and its own count
  const auto pick = [&](int shift) {
    __syncthreads();
    if (tid == 0) {
      uint32_t cum = 0u, b = 0u;
      for (; b < 255u && cum + hist[b] < need; ++b) cum += hist[b];
      s_pick[0] = b;
      s_pick[1] = need - cum;
      s_pick[2] = hist[b];
    }
    __syncthreads();
    need = s_pick[1];
    at_T = s_pick[2];
    const uint32_t byte = s_pick[0] << shift;
    __syncthreads();
    return byte;
  };
  for (int shift = 24; shift >= 0; shift -= 8) {
    hist[tid] = 0u;
    __syncthreads();
    visit_runs<E>(pts, boxes, n, q, reach, [&](int, float d2, bool valid) {
      const uint32_t u = __float_as_uint(d2);
      if (valid && (u & mask) == prefix) atomicAdd(&hist[(u >> shift) & 255u], 1u);
    });
    prefix |= pick(shift);
    mask |= 255u << shift;
    // no entry needed lies beyond the counter's range
    reach = fminf(reach, __uint_as_float(min(prefix | ~mask, 0x7f800000u)));
  }
  // rank of the last index taken at distance T, when not all are: radix
  // select on j
  const uint32_t T = prefix;
  uint32_t jpre = 0u, jmask = 0u;
  if (need == at_T) {
    jpre = ~0u;
  } else {
    for (int shift = 24; shift >= 0; shift -= 8) {
      hist[tid] = 0u;
      __syncthreads();
      visit_runs<E>(pts, boxes, n, q, reach, [&](int c, float d2, bool valid) {
        if (valid && __float_as_uint(d2) == T) {
          const uint32_t j = (uint32_t)qord[c];
          if ((j & jmask) == jpre) atomicAdd(&hist[(j >> shift) & 255u], 1u);
        }
      });
      jpre |= pick(shift);
      jmask |= 255u << shift;
    }
  }
  // exactly w keys are at most (T, jpre): collect and sort them
  const uint64_t last = ((uint64_t)T << 32) | jpre;
  if (tid == 0) s_at = 0;
  __syncthreads();
  visit_runs<E>(pts, boxes, n, q, reach, [&](int c, float d2, bool valid) {
    const uint64_t key = row_key(d2, valid ? qord[c] : -1);
    if (valid && key <= last) {
      const int at = atomicAdd(&s_at, 1);
      if (at < w) grouped[at] = key;
    }
  });
  int P = 1;
  while (P < w) P <<= 1;
  __syncthreads();
  for (int x = min(s_at, w) + tid; x < P; x += kBlock) grouped[x] = ~0ull;
  __syncthreads();
  for (int size = 2; size <= P; size <<= 1)
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int x = tid; x < P / 2; x += kBlock) {
        const int lo = 2 * x - (x & (stride - 1));
        const int hi = lo + stride;
        const bool up = (lo & size) == 0;
        const uint64_t a = grouped[lo], b = grouped[hi];
        if ((a > b) == up) {
          grouped[lo] = b;
          grouped[hi] = a;
        }
      }
      __syncthreads();
    }
  for (int x = tid; x < w; x += kBlock) row[x] = grouped[x];
}

// Neighbour rows: row p of a job = the first w embedded points of its
// embedding in ascending (d2, j) order from the point at visiting position
// p, as keys (d2 bits, j); entries past n_e are ~0.
//
// One workgroup per run of consecutive positions.  The w-th distance changes
// little from one position to the next, so each row starts from a threshold
// above the previous row's w-th distance, aimed at 1.5 w points by the
// measured growth of their number: one pass over the runs of 64 points whose
// box reaches within it collects the candidates (bound by that pass: 2E
// operations and one load per coordinate for each point visited), and only a
// row whose threshold caught fewer than w or more than fit repeats it with
// another (1.04 passes per row at E = 2, 1.1 at E = 3 and 4, 1.3 to 1.7 at
// E = 10).  The candidates are then ordered by bucket of d2
// and by comparison within a bucket, a tenth of the work of a sorting
// network at w = 1024.  The keys are regrouped in place through registers:
// a second array left a third of the wavefronts (10^5 rows of 10^4 points,
// E = 1: 0.98 against 0.66 ms).  Building two or four rows per pass, to load
// the points once for them, was 15-25% slower: their thresholds are missed
// more often together, and their candidates take LDS from other workgroups.
// Rows among repeated values (more points at one distance than fit, or than
// are worth comparing) are left to k_rows_repeats, and so are rows whose nearest
// points lie in the runs of one wavefront, more than its segment holds.
//
// Minimum wavefronts per SIMD: 6 at small E and 5 from E = 6 on, each within
// 3% of the other and 4-13% faster than 4 or 7.
template <int E>
__global__ __launch_bounds__(kBlock)
__attribute__((amdgpu_waves_per_eu(E < 6 ? 6 : 5, 8))) void k_rows(
    const RowJob* __restrict__ jobs, int per_block, const float* __restrict__ pts_pool,
    const float* __restrict__ box_pool, const int32_t* __restrict__ qord_pool,
    uint64_t* __restrict__ row_pool, RowTodo* __restrict__ todo, int* __restrict__ todo_n) {
  extern __shared__ uint64_t row_lds[];
  __shared__ int s_n[kWaves], s_wave[kWaves], s_full[kWaves];
  __shared__ float s_t;
  const RowJob J = jobs[blockIdx.y];
  const int n = J.n_e;
  const int p0 = (int)blockIdx.x * per_block;
  if (p0 >= n) return;                            // the whole workgroup
  const int w = min(J.w, n);
  const int seg = row_segment(J.w);
  uint64_t* __restrict__ cand = row_lds;
  uint64_t* __restrict__ grouped = row_lds;       // over the segments
  uint32_t* __restrict__ hist = reinterpret_cast<uint32_t*>(row_lds + kWaves * seg);
  const float* __restrict__ pts = pts_pool + J.pts_off;
  const float* __restrict__ boxes = box_pool + J.box_off;
  const int32_t* __restrict__ qord = qord_pool + J.qord_off;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  // the number of points within t grows about like t^growth; from the last rows
  float growth = 0.5f * E;
  float t_next = -1.f;
  bool repeats = false;                            // the last row was left

  for (int p = p0; p < min(p0 + per_block, n); ++p) {
    float q[E];
#pragma unroll
    for (int k = 0; k < E; ++k) q[k] = pts[(int64_t)k * n + p];
    uint64_t* __restrict__ row = row_pool + J.out_off + (int64_t)p * J.w;
    const auto order_bound = [&] { return order_reach<E>(pts, n, w, p, q, s_n); };
    float t = repeats && (p & 7) ? 0.f : t_next < 0.f ? order_bound() : t_next;
    // thresholds known to catch too few / enough, but more than fit
    float t_few = -1.f, t_many = __builtin_inff();
    int total = 0;
    bool done = false;
    for (int attempt = 0; attempt < (repeats && (p & 7) ? 0 : 16) && !done; ++attempt) {
      const float scale = t > 0.f ? (float)kRowBuckets / t : 0.f;
      for (int b = tid; b < kRowBuckets; b += kBlock) hist[b] = 0u;
      __syncthreads();
      int mine = 0;
      visit_runs<E>(pts, boxes, n, q, t, [&](int c, float d2, bool valid) {
        const bool keep = valid && d2 <= t;
        const uint64_t m = __builtin_amdgcn_ballot_w64(keep);
        if (m) {
          const int at = mine + __popcll(m & below);
          if (keep && at < seg) {
            const uint64_t key = row_key(d2, qord[c]);
            cand[wave * seg + at] = key;
            atomicAdd(&hist[row_bucket(key, scale, 0u)], 1u);
          }
          mine += __popcll(m);
        }
      });
      if (lane == 0) s_n[wave] = mine;
      __syncthreads();
      bool over = false;
      total = 0;
#pragma unroll
      for (int v = 0; v < kWaves; ++v) {
        over |= s_n[v] > seg;
        total += s_n[v];
      }
      // one wavefront's share is full before there are w: so it is for every
      // larger threshold, and this one bounds nothing
      if (over && total < w) break;
      if (total < w || over) {
        (over ? t_many : t_few) = t;
        // by the power law, else into the bracket
        float to = t * exp2f(log2f(kRowTarget * (float)w / (float)max(total, 1)) / growth);
        if (attempt >= 2 || !(to > t_few && to < t_many)) {
          if (!(t_many < __builtin_inff()))
            to = order_bound();
          else
            to = t_few > 0.f ? sqrtf(t_few) * sqrtf(t_many) : 0.5f * t_many;
        }
        t = to;
        if (!(t > t_few && t < t_many)) break;
      } else {
        done = true;
      }
    }
    int crowded = 0;
    if (done) {
      float scale = t > 0.f ? (float)kRowBuckets / t : 0.f;
      const uint32_t t_bits = __float_as_uint(t);
      const uint32_t base = t_bits > (32u << 23) ? t_bits - (32u << 23) : 0u;
      // the keys into registers, spread over the threads
      int before[kWaves + 1];
      before[0] = 0;
#pragma unroll
      for (int v = 0; v < kWaves; ++v) before[v + 1] = before[v] + s_n[v];
      uint64_t mine[kRowPerThread];
#pragma unroll
      for (int u = 0; u < kRowPerThread; ++u) {
        const int x = u * kBlock + tid;
        if (u * kBlock >= total) break;
        int at = x;
#pragma unroll
        for (int v = 1; v < kWaves; ++v)
          if (x >= before[v]) at = v * seg + x - before[v];
        mine[u] = x < total ? cand[at] : 0ull;
      }
      for (;;) {
        // exclusive prefix over the buckets: four per thread
        constexpr int per = kRowBuckets / kBlock;
        uint32_t h[per], sum = 0;
#pragma unroll
        for (int u = 0; u < per; ++u) {
          h[u] = hist[tid * per + u];
          sum += h[u];
        }
        uint32_t inc = sum;
#pragma unroll
        for (int s = 1; s < 64; s <<= 1) {
          const uint32_t y = __shfl_up(inc, s, 64);
          if (lane >= s) inc += y;
        }
        if (lane == 63) s_wave[wave] = (int)inc;
        __syncthreads();
        uint32_t at = inc - sum;
        for (int v = 0; v < wave; ++v) at += (uint32_t)s_wave[v];
        // a bucket of the row too full to be ordered by comparison
        const uint32_t most = scale < 0.f ? kRowMost : kRowCrowd;
        int full = 0;
#pragma unroll
        for (int u = 0; u < per; ++u) {
          if (h[u] > most && (int)at < w) full = 1;
          hist[tid * per + u] = at;
          at += h[u];
        }
        const bool any_full = __builtin_amdgcn_ballot_w64(full) != 0;
        if (lane == 0) s_full[wave] = any_full ? 1 : 0;
        __syncthreads();
        crowded = s_full[0] | s_full[1] | s_full[2] | s_full[3];
        if (!crowded || scale < 0.f) break;
        // (distances of very different sizes: by octave)
        scale = -1.f;
        for (int b = tid; b < kRowBuckets; b += kBlock) hist[b] = 0u;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kRowPerThread; ++u) {
          if (u * kBlock >= total) break;
          if (u * kBlock + tid < total) atomicAdd(&hist[row_bucket(mine[u], scale, base)], 1u);
        }
        __syncthreads();
      }
      // grouped by bucket; afterwards hist[b] is the end of bucket b
#pragma unroll
      for (int u = 0; u < kRowPerThread; ++u) {
        if (u * kBlock >= total) break;
        if (u * kBlock + tid < total)
          grouped[atomicAdd(&hist[row_bucket(mine[u], scale, base)], 1u)] = mine[u];
      }
      __syncthreads();
      if (!crowded) {
        for (int x = tid; x < total; x += kBlock) {
          const uint64_t key = grouped[x];
          const int b = row_bucket(key, scale, base);
          const int lo = b ? (int)hist[b - 1] : 0, hi = (int)hist[b];
          if (lo >= w) continue;
          int r = lo;
          for (int y = lo; y < hi; ++y) r += grouped[y] < key ? 1 : 0;
          if (r < w) row[r] = key;
          if (r == w - 1) s_t = __uint_as_float((uint32_t)(key >> 32));
        }
        __syncthreads();
        const float s = s_t;
        if (total > w && t > 1.0001f * s && s > 0.f)
          growth += 0.3f * (fminf(2.f * E, fmaxf(0.5f, log2f((float)total / (float)w) /
                                                           log2f(t / s))) - growth);
      }
    }
    if (!done || crowded) {
      // left to k_rows_repeats; the rows after it go there unseen, but for
      // every eighth
      if (tid == 0) {
        const int at = atomicAdd(todo_n, 1);
        todo[at] = {(int)blockIdx.y, p, done ? t : t_many, 0};
      }
      repeats = true;
      t_next = -1.f;
    } else {
      for (int x = w + tid; x < J.w; x += kBlock) row[x] = ~0ull;
      repeats = false;
      t_next = s_t * exp2f(log2f(kRowTarget) / growth);
    }
  }
}

// The rows k_rows has left (todo_n of them), by distance or by selection.
template <int E>
__global__ __launch_bounds__(kBlock) void k_rows_repeats(
    const RowJob* __restrict__ jobs, const RowTodo* __restrict__ todo,
    const int* __restrict__ todo_n, const float* __restrict__ pts_pool,
    const float* __restrict__ box_pool, const int32_t* __restrict__ qord_pool,
    uint64_t* __restrict__ row_pool) {
  extern __shared__ uint64_t row_lds[];
  __shared__ int s_n[kWaves];
  const int count = *todo_n;
  for (int x = blockIdx.x; x < count; x += gridDim.x) {
    const RowTodo D = todo[x];
    const RowJob J = jobs[D.job];
    const int n = J.n_e, w = min(J.w, n);
    const int words = kWaves * row_segment(J.w) * 2;
    const float* __restrict__ pts = pts_pool + J.pts_off;
    const float* __restrict__ boxes = box_pool + J.box_off;
    const int32_t* __restrict__ qord = qord_pool + J.qord_off;
    uint64_t* __restrict__ row = row_pool + J.out_off + (int64_t)D.p * J.w;
    float q[E];
#pragma unroll
    for (int k = 0; k < E; ++k) q[k] = pts[(int64_t)k * n + D.p];
    const float reach =
        D.reach < __builtin_inff() ? D.reach : order_reach<E>(pts, n, w, D.p, q, s_n);
    if (!row_by_level<E>(pts, boxes, qord, n, w, q, reach, reinterpret_cast<uint32_t*>(row_lds),
                         words, row)) {
      __syncthreads();
      row_by_select<E>(pts, boxes, qord, n, w, q, reach, row_lds,
                       reinterpret_cast<uint32_t*>(row_lds + kWaves * row_segment(J.w)), row);
    }
    for (int y = w + (int)threadIdx.x; y < J.w; y += kBlock) row[y] = ~0ull;
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// the walk: 64 libraries per wavefront
// ---------------------------------------------------------------------------

// Transpose of a 64 x 64 bit matrix, row l in lane l: afterwards bit e of
// lane r is what bit r of lane e was.  Blocks of 32, 16, ..., 1 are
// exchanged between lanes that far apart; 32 and 16 with the half- and
// row-swap instructions, 8 and below within rows of 16 lanes (DPP).
struct BitTranspose {
  uint32_t sel16, sel8, rot4, m4, rot2, m2, rot1, m1;
  __device__ __forceinline__ explicit BitTranspose(int lane) {
    sel16 = (lane & 16) ? 0x07060302u : 0x05040100u;   // bytes of (odd row, even row)
    sel8 = (lane & 8) ? 0x03070105u : 0x06020400u;     // bytes of (partner, own)
    rot4 = (lane & 4) ? 4u : 28u;
    m4 = (lane & 4) ? 0xf0f0f0f0u : 0x0f0f0f0fu;
    rot2 = (lane & 2) ? 2u : 30u;
    m2 = (lane & 2) ? 0xccccccccu : 0x33333333u;
    rot1 = (lane & 1) ? 1u : 31u;
    m1 = (lane & 1) ? 0xaaaaaaaau : 0x55555555u;
  }
  template <int CTRL>
  __device__ __forceinline__ static uint32_t dpp(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, true);
  }
  __device__ __forceinline__ uint32_t within(uint32_t x) const {
    // rows of 16 lanes: even rows keep their low halves and take the odd
    // row's low halves above them, odd rows the high halves likewise
    const auto s = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    x = __builtin_amdgcn_perm(s[1], s[0], sel16);
    // 8: row_ror:8 pairs lanes l and l ^ 8
    x = __builtin_amdgcn_perm(dpp<0x128>(x), x, sel8);
    // 4: mirror within 8, then within 4
    uint32_t y = dpp<0x1b>(dpp<0x141>(x));
    y = __builtin_amdgcn_alignbit(y, y, rot4);
    x = (x & m4) | (y & ~m4);
    y = dpp<0x4e>(x);                                  // quad_perm 2,3,0,1
    y = __builtin_amdgcn_alignbit(y, y, rot2);
    x = (x & m2) | (y & ~m2);
    y = dpp<0xb1>(x);                                  // quad_perm 1,0,3,2
    y = __builtin_amdgcn_alignbit(y, y, rot1);
    return (x & m1) | (y & ~m1);
  }
  __device__ __forceinline__ uint64_t operator()(uint64_t m) const {
    const auto s = __builtin_amdgcn_permlane32_swap((uint32_t)m, (uint32_t)(m >> 32), false,
                                                    false);
    return (uint64_t)within(s[0]) | ((uint64_t)within(s[1]) << 32);
  }
};

// Quotient x / y of finite x >= 0, y > 0 with r = fl(1 / y): x r corrected
// twice by its exact remainder, which gives the correctly rounded quotient
// (Markstein, "Computation of elementary functions on the IBM RISC
// System/6000 processor", 1990) as long as neither the quotient nor a
// remainder underflows; smaller x take the division.
__device__ __forceinline__ double quotient(double x, double y, double r) {
  double q = x * r;
  q = __builtin_fma(__builtin_fma(-q, y, x), r, q);
  q = __builtin_fma(__builtin_fma(-q, y, x), r, q);
  if (__builtin_expect(!(x > 0x1p-900), 0)) {
    asm volatile("");                              // a branch, not a select
    q = x / y;
  }
  return q;
}

// LDS of one wavefront of the walk: the chunk's values by entry, then the
// accepted ones by rank and lane.
template <int E, bool KEYS>
struct WalkLds {
  static constexpr int K = E + 1;
  double chunk[KEYS ? 1 : 2][64];
  double slot[KEYS ? 1 : 2][K][64];
};

// One item: the queries at visiting positions [tile * per, (tile + 1) * per)
// of one embedding against the (at most 64) libraries of one group, lane l
// of each wavefront holding library l.  Per query the row is read 64 entries
// at a time; each lane reads one entry and its membership word (bit l:
// library l holds the point; 0 for excluded points), and the transposed
// words give every library its members among the 64 entries in row order.
// Lanes take their lowest set bits until they hold E+1 neighbours; then the
// prediction is formed with simplex_weights' operations (KEYS: the
// neighbours' keys are written instead).  A library that finds fewer than
// E+1 in the whole row (its rows were cut at w entries) is searched in full
// by the wavefront (about one query in 10^7 by the planner's row length).
//
// Bound by the FP64 exponentials of the predictions (E+1 each), and below
// that by instruction issue: a chunk costs about 31 instructions for the
// transpose, and a member about 18 to take out.
template <int E, bool KEYS>
__global__ __launch_bounds__(kBlock) void k_walk(
    const WalkGroup* __restrict__ groups, const RowJob* __restrict__ embs,
    const Item* __restrict__ items, int per,
    const uint64_t* __restrict__ mask_pool, const uint64_t* __restrict__ row_pool,
    const int32_t* __restrict__ qord_pool, const float* __restrict__ emb_pool,
    const double* __restrict__ tgt_pool, double* __restrict__ out, int excl, int query_set) {
  constexpr int K = E + 1;
  __shared__ WalkLds<E, KEYS> s_lds[kWaves];
  const Item I = items[xcd_item(blockIdx.x, gridDim.x)];
  const WalkGroup G = groups[I.rz];
  const RowJob J = embs[G.emb];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  WalkLds<E, KEYS>& lds = s_lds[wave];
  const uint64_t* __restrict__ masks = mask_pool + G.mask_off;
  const int32_t* __restrict__ qord = qord_pool + J.qord_off;
  const double* __restrict__ tgt = tgt_pool + G.tgt_off;
  const bool mine = lane < G.n_lib;
  const BitTranspose transpose(lane);
  const int sub = (per + kWaves - 1) / kWaves;
  const int pa = I.tile * per + wave * sub;
  const int pb = min(min(pa + sub, I.tile * per + per), J.n_e);
  if (pa >= pb) return;                            // no barrier below

  // Software pipeline over the queries: the first chunk of the next query's
  // row is requested while this query's is taken apart, and its membership
  // words and targets before this query's prediction.
  int i = qord[pa];
  const uint64_t* __restrict__ row = row_pool + J.out_off + (int64_t)pa * J.w;
  uint64_t key = row[lane];
  uint64_t m = 0;
  double tv = 0.0;
  // membership word and target of a row entry (0 for excluded points)
  const auto entry = [&](uint64_t k, int self, uint64_t& mm, double& tt) {
    const int j = (int)(uint32_t)k;
    mm = 0;
    if (j >= 0) {
      const int gap = j > self ? j - self : self - j;
      if (gap > excl) mm = masks[j];
      if (!KEYS) tt = tgt[j];
    }
  };
  entry(key, i, m, tv);
  for (int p = pa; p < pb; ++p) {
    const int p1 = min(p + 1, pb - 1);
    const int i_next = qord[p1];
    const uint64_t* __restrict__ row_next = row_pool + J.out_off + (int64_t)p1 * J.w;
    const uint64_t key_next = row_next[lane];
    bool active = mine;
    if (query_set) active = active && ((masks[i] >> lane) & 1ull);
    int cnt = active ? 0 : K;
    for (int c = 0;;) {
      const bool more = c + 1 < G.chunks;
      const uint64_t key_c = row[(more ? c + 1 : c) * 64 + lane];
      wave_sync();
      if (KEYS) {
        lds.chunk[0][lane] = __longlong_as_double((long long)key);
      } else {
        lds.chunk[0][lane] = sqrt((double)__uint_as_float((uint32_t)(key >> 32)));
        lds.chunk[KEYS ? 0 : 1][lane] = tv;
      }
      uint64_t bits = transpose(m);
      if (cnt >= K) bits = 0;
      wave_sync();
      while (__builtin_amdgcn_ballot_w64(bits != 0)) {
        if (bits) {
          const int e = __builtin_ctzll(bits);
          bits &= bits - 1ull;
          lds.slot[0][cnt][lane] = lds.chunk[0][e];
          if (!KEYS) lds.slot[KEYS ? 0 : 1][cnt][lane] = lds.chunk[KEYS ? 0 : 1][e];
          if (++cnt == K) bits = 0;
        }
      }
      if (!more || !__builtin_amdgcn_ballot_w64(cnt < K)) break;
      ++c;
      key = key_c;
      entry(key, i, m, tv);
    }
    key = key_next;
    entry(key, i_next, m, tv);
    // libraries whose row ran short: the wavefront looks through the whole
    // library, each lane keeping the K smallest keys of its share, and takes
    // the K smallest of all of them one by one
    uint64_t shortfall = __builtin_amdgcn_ballot_w64(cnt < K);
    while (shortfall) {
      const int l = __builtin_ctzll(shortfall);
      shortfall &= shortfall - 1ull;
      const float* __restrict__ emb = emb_pool + J.emb_off;
      float q[E];
#pragma unroll
      for (int k = 0; k < E; ++k) q[k] = emb[(int64_t)i * J.stride + k];
      double best[K];
#pragma unroll
      for (int t = 0; t < K; ++t) best[t] = empty_key();
      constexpr int kAhead = 8;                    // membership words in flight
      for (int j0 = 0; j0 < J.n_e; j0 += 64 * kAhead) {
        uint64_t m[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) m[u] = masks[min(j0 + u * 64 + lane, J.n_e - 1)];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
          const int j = j0 + u * 64 + lane;
          const int gap = j > i ? j - i : i - j;
          if (j < J.n_e && gap > excl && ((m[u] >> l) & 1ull))
            insert_key<K>(best, make_key(sqdist<E>(q, emb + (int64_t)j * J.stride), j));
        }
      }
#pragma unroll 1
      for (int t = 0; t < K; ++t) {
        double lo = best[0];
#pragma unroll
        for (int s = 32; s > 0; s >>= 1) {
          const double o = __hiloint2double(__shfl_xor(__double2hiint(lo), s, 64),
                                            __shfl_xor(__double2loint(lo), s, 64));
          lo = kmin(lo, o);
        }
        if (__double_as_longlong(best[0]) == __double_as_longlong(lo)) {
#pragma unroll
          for (int u = 0; u + 1 < K; ++u) best[u] = best[u + 1];
          best[K - 1] = empty_key();
        }
        if (lane == l) {
          // (an empty place, left where the distances are NaN: point 0)
          const int j = max(key_j(lo), 0);
          if (KEYS) {
            lds.slot[0][t][lane] = make_key(key_d2(lo), j);
          } else {
            lds.slot[0][t][lane] = sqrt((double)key_d2(lo));
            lds.slot[KEYS ? 0 : 1][t][lane] = tgt[j];
          }
        }
      }
    }
    if (active) {
      if constexpr (KEYS) {
        double* __restrict__ o =
            out + G.out_off + (int64_t)(query_set ? i : p) * (K * G.n_lib) + lane;
#pragma unroll
        for (int t = 0; t < K; ++t) o[t * G.n_lib] = lds.slot[0][t][lane];
      } else {
        // the operations of simplex_weights and of the weighted sum
        double u[K];
        const double d0 = lds.slot[0][0][lane];
        if (d0 > 0.0) {
          const double r = 1.0 / d0;
#pragma unroll
          for (int t = 0; t < K; ++t) u[t] = exp(-quotient(lds.slot[0][t][lane], d0, r));
        } else {
#pragma unroll
          for (int t = 0; t < K; ++t) u[t] = lds.slot[0][t][lane] == 0.0 ? 1.0 : 0.0;
        }
        double su = 0.0;
#pragma unroll
        for (int t = 0; t < K; ++t) su += u[t];
        const double rs = 1.0 / su;
        double pred = 0.0;
#pragma unroll
        for (int t = 0; t < K; ++t)
          pred += quotient(u[t], su, rs) * lds.slot[KEYS ? 0 : 1][t][lane];
        out[G.out_off + (int64_t)(query_set ? i : p) * G.n_lib + lane] = pred;
      }
    }
    i = i_next;
    row = row_next;
  }
}

// Moments of one query tile of a walked realization from its predictions:
// the same queries per lane, operations and merge order as crossmap_item.
template <int Q>
__global__ __launch_bounds__(kBlock) void k_walk_moments(
    const Realization* __restrict__ rzs, const WalkOut* __restrict__ where,
    const Item* __restrict__ items, const double* __restrict__ pred,
    const int32_t* __restrict__ pj_pool, const int32_t* __restrict__ qord_pool,
    const double* __restrict__ tgt_pool, Moments* __restrict__ partial, int query_set) {
  __shared__ Moments red[kBlock];
  const Item I = items[xcd_item(blockIdx.x, gridDim.x)];
  const Realization R = rzs[I.rz];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const double* __restrict__ tgt = tgt_pool + R.tgt_off + (int64_t)(R.E - 1) * R.tau;
  const int32_t* __restrict__ q = query_set ? pj_pool + R.pj_off : qord_pool + R.qord_off;
  const WalkOut W = where[I.rz];
  const double* __restrict__ pr = pred + W.off;
  Moments mo = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int m = 0; m < Q; ++m) {
    const int qq = I.tile * (kBlock * Q) + wave * (64 * Q) + m * 64 + lane;
    if (qq < R.n_query) {
      const int i = q[qq];
      mom_add(mo, tgt[i], pr[(int64_t)(query_set ? i : qq) * W.stride]);
    }
  }
  red[tid] = mo;
  __syncthreads();
#pragma unroll
  for (int s = kBlock / 2; s > 0; s >>= 1) {
    if (tid < s) red[tid] = mom_merge(red[tid], red[tid + s]);
    __syncthreads();
  }
  if (tid == 0) partial[R.slot_base + I.tile] = red[0];
}

// Causal matrix: one query tile of up to 16 libraries of a walk group, whose
// neighbours the walk has left as keys.  Wavefront v takes the libraries
// 4 v .. 4 v + 3 of the sixteen, two at a time: lanes 0..31 one of them, lanes
// 32..63 the other, each lane two neighbouring targets, and goes through the
// tile's queries in order.
//
// Bound by the vector memory path: a load of one 8-byte value per lane takes
// 16 of its cycles like one of 16 bytes, so two targets per lane halve them
// (64 series, N = 20000, E = 4, r = 10: 27.8 ms with one target per lane and
// one library at a time, 18.4 now).  The neighbours of one query in different
// libraries are mostly the same few points, so two thirds of the loads hit in
// L1 (a workgroup per library read 360 GB from L2; 23 ms); a fourth wavefront
// per SIMD, with the earlier runs' sums in memory, gained nothing for the L1
// it took.  The observed side of the sums is formed once for the four
// libraries.
//
// Sums as in multi_target_block, in its order: over the run of 64 Q queries
// of each of its four wavefronts, then the four runs' sums in order.
template <int E>
struct GroupLds {
  static constexpr int K = E + 1;
  static constexpr int kLibs = kMultiLibs / kWaves;  // libraries of one wavefront
  static constexpr int kSet = 128 / kLibs;           // queries staged together
  double w[kLibs][K][kSet];
  uint32_t row[kLibs][K][kSet];                      // byte offsets of the neighbours' rows
  uint32_t qrow[kSet];
};

template <int E, int Q>
__global__ __launch_bounds__(kBlock) void k_multi_group(
    const Realization* __restrict__ rzs, const int32_t* __restrict__ self_of,
    const WalkGroup* __restrict__ groups, const WalkLib* __restrict__ libs,
    const Item* __restrict__ items, const double* __restrict__ keys,
    const int32_t* __restrict__ qord_pool, const double* __restrict__ tt, int m_series,
    Sums* __restrict__ partial) {
  constexpr int K = E + 1;
  constexpr int kLibs = GroupLds<E>::kLibs;
  constexpr int kSet = GroupLds<E>::kSet;
  __shared__ GroupLds<E> s_lds[kWaves];
  const Item I = items[xcd_item(blockIdx.x, gridDim.x)];
  const WalkGroup G = groups[I.rz >> 2];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l0 = (I.rz & 3) * kMultiLibs + wave * kLibs;   // first library of the wavefront
  if (l0 >= G.n_lib) return;                       // no barrier below
  const int nl = min(kLibs, G.n_lib - l0);
  const Realization R = rzs[libs[G.lib_first + l0].rz];   // shape shared by the group
  const int self = self_of[libs[G.lib_first + l0].rz];
  GroupLds<E>& lds = s_lds[wave];
  const int mp = target_stride(m_series);
  const double* __restrict__ T = tt + (int64_t)(E - 1) * R.tau * mp;
  const char* __restrict__ Tc = reinterpret_cast<const char*>(T);
  const int32_t* __restrict__ qord = qord_pool + R.qord_off;
  const double* __restrict__ kp = keys + G.out_off + l0;
  const int half = lane >> 5;                      // library of the pair
  constexpr int kPairs = kLibs / 2;
  constexpr int kT = 2;                            // targets per lane

  for (int b0 = 0; b0 < m_series; b0 += 64) {
    const int b = b0 + kT * (lane & 31);                   // (mp is even: both columns exist)
    const uint32_t lb = b < m_series ? (uint32_t)b * 8u : 0u;
    const auto at = [&](uint32_t row_bytes) {
      return *reinterpret_cast<const double2*>(Tc + (row_bytes + lb));
    };
    const double2 sh = at(0u);
    const double shift[kT] = {sh.x, sh.y};
    // the sums of the runs before this one: n and the observed side, then
    // each library's predicted side
    double n_all = 0.0, so_all[kT], soo_all[kT];
    double sp_all[kPairs][kT], spp_all[kPairs][kT], sop_all[kPairs][kT];
    double mno[kT], mxo[kT], mnp[kPairs][kT], mxp[kPairs][kT];
#pragma unroll
    for (int x = 0; x < kT; ++x) {
      mno[x] = __builtin_inf();
      mxo[x] = -__builtin_inf();
#pragma unroll
      for (int h = 0; h < kPairs; ++h) {
        mnp[h][x] = __builtin_inf();
        mxp[h][x] = -__builtin_inf();
      }
    }
    for (int run = 0; run < kWaves; ++run) {
      double n_run = 0.0, so[kT] = {0.0, 0.0}, soo[kT] = {0.0, 0.0};
      double sp[kPairs][kT], spp[kPairs][kT], sop[kPairs][kT];
#pragma unroll
      for (int h = 0; h < kPairs; ++h)
#pragma unroll
        for (int x = 0; x < kT; ++x) sp[h][x] = spp[h][x] = sop[h][x] = 0.0;
      const int q_run = I.tile * (kBlock * Q) + run * (64 * Q);
      for (int s0 = 0; s0 < 64 * Q; s0 += kSet) {
        const int nq = min(kSet, R.n_query - (q_run + s0));
        if (nq <= 0) break;
        // stage, lane by (library, query); past the last library, the last one
        // again
        const int sub = lane & (kSet - 1);
        const int p = q_run + s0 + min(sub, nq - 1);
        wave_sync();
        if (lane < kSet) lds.qrow[sub] = (uint32_t)(qord[p] * mp) * 8u;
#pragma unroll
        for (int h = 0; h < kLibs * kSet / 64; ++h) {
          const int u = h * (64 / kSet) + lane / kSet;
          // the operations of stage_weights
          double v[K], su = 0.0;
          int32_t j[K];
#pragma unroll
          for (int t = 0; t < K; ++t) {
            const double key = kp[((int64_t)p * K + t) * G.n_lib + min(u, nl - 1)];
            v[t] = sqrt((double)key_d2(key));
            j[t] = key_j(key);
          }
          const double d0 = v[0];
          if (d0 > 0.0) {
            const double r = 1.0 / d0;
#pragma unroll
            for (int t = 0; t < K; ++t) {
              v[t] = exp(-quotient(v[t], d0, r));
              su += v[t];
            }
          } else {
#pragma unroll
            for (int t = 0; t < K; ++t) {
              v[t] = v[t] == 0.0 ? 1.0 : 0.0;
              su += v[t];
            }
          }
          const double rs = 1.0 / su;
#pragma unroll
          for (int t = 0; t < K; ++t) {
            lds.w[u][t][sub] = quotient(v[t], su, rs);
            lds.row[u][t][sub] = (uint32_t)(j[t] * mp) * 8u;
          }
        }
        wave_sync();
        n_run += (double)nq;
        for (int q = 0; q < nq; ++q) {
          const double2 ov = at(lds.qrow[q]);
          const double o[kT] = {ov.x, ov.y};
          double a[kT];
#pragma unroll
          for (int x = 0; x < kT; ++x) {
            a[x] = o[x] - shift[x];
            so[x] += a[x];
            soo[x] = fma(a[x], a[x], soo[x]);
            mno[x] = kmin(mno[x], o[x]);
            mxo[x] = kmax(mxo[x], o[x]);
          }
#pragma unroll
          for (int h = 0; h < kPairs; ++h) {
            if (2 * h >= nl) break;
            const int u = 2 * h + half;
            double2 v[K];
#pragma unroll
            for (int t = 0; t < K; ++t) v[t] = at(lds.row[u][t][q]);
            double wt = lds.w[u][0][q];
            double pred[kT] = {wt * v[0].x, wt * v[0].y};
#pragma unroll
            for (int t = 1; t < K; ++t) {
              wt = lds.w[u][t][q];
              pred[0] = fma(wt, v[t].x, pred[0]);
              pred[1] = fma(wt, v[t].y, pred[1]);
            }
#pragma unroll
            for (int x = 0; x < kT; ++x) {
              const double d = pred[x] - shift[x];
              sp[h][x] += d;
              spp[h][x] = fma(d, d, spp[h][x]);
              sop[h][x] = fma(a[x], d, sop[h][x]);
              mnp[h][x] = kmin(mnp[h][x], pred[x]);
              mxp[h][x] = kmax(mxp[h][x], pred[x]);
            }
          }
        }
      }
      // the first run's sums are taken as they are, the others' added
      n_all = run == 0 ? n_run : n_all + n_run;
#pragma unroll
      for (int x = 0; x < kT; ++x) {
        so_all[x] = run == 0 ? so[x] : so_all[x] + so[x];
        soo_all[x] = run == 0 ? soo[x] : soo_all[x] + soo[x];
#pragma unroll
        for (int h = 0; h < kPairs; ++h) {
          sp_all[h][x] = run == 0 ? sp[h][x] : sp_all[h][x] + sp[h][x];
          spp_all[h][x] = run == 0 ? spp[h][x] : spp_all[h][x] + spp[h][x];
          sop_all[h][x] = run == 0 ? sop[h][x] : sop_all[h][x] + sop[h][x];
        }
      }
    }
#pragma unroll
    for (int h = 0; h < kPairs; ++h) {
      const int u = 2 * h + half;
      if (u >= nl) continue;
      const int64_t slot = rzs[libs[G.lib_first + l0 + u].rz].slot_base;
#pragma unroll
      for (int x = 0; x < kT; ++x) {
        if (b + x >= m_series || b + x == self) continue;
        Sums s;
        s.v[0] = n_all;
        s.v[1] = so_all[x];
        s.v[2] = sp_all[h][x];
        s.v[3] = soo_all[x];
        s.v[4] = spp_all[h][x];
        s.v[5] = sop_all[h][x];
        s.v[6] = mno[x];
        s.v[7] = mxo[x];
        s.v[8] = mnp[h][x];
        s.v[9] = mxp[h][x];
        partial[(slot + I.tile) * m_series + b + x] = s;
      }
    }
  }
}

// Causal matrix, few items or library-point queries (each library has its
// own): one query tile of a walked realization, its neighbours read from the
// walk's keys instead of searched; then the
// per-target stage of crossmap_multi_item.
template <int E, int Q>
__global__ __launch_bounds__(kBlock) void k_multi_keys(
    const Realization* __restrict__ rzs, const int32_t* __restrict__ self_of,
    const WalkOut* __restrict__ where, const Item* __restrict__ items,
    const double* __restrict__ keys, const int32_t* __restrict__ pj_pool,
    const int32_t* __restrict__ qord_pool, const double* __restrict__ tt, int m_series,
    Sums* __restrict__ partial, int query_set) {
  __shared__ __align__(16) unsigned char lds[MultiLds<E>::kBytes];
  const Item I = items[xcd_item(blockIdx.x, gridDim.x)];
  const Realization R = rzs[I.rz];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int32_t* __restrict__ q = query_set ? pj_pool + R.pj_off : qord_pool + R.qord_off;
  const WalkOut W = where[I.rz];
  const double* __restrict__ k = keys + W.off;
  ScanState<E, Q, kKeepSelf> S;
#pragma unroll
  for (int m = 0; m < Q; ++m) {
    const int qq = I.tile * (kBlock * Q) + wave * (64 * Q) + m * 64 + lane;
    const bool valid = qq < R.n_query;
    const int i = valid ? q[qq] : 0;
    const int at = query_set ? i : (valid ? qq : 0);
    S.qi[m] = valid ? i : -1;
#pragma unroll
    for (int t = 0; t < E + 1; ++t) S.key[m][t] = k[((int64_t)at * (E + 1) + t) * W.stride];
  }
  multi_targets<E, Q, kKeepSelf>(S, R, I.tile, tt, m_series, self_of[I.rz], partial, lds);
}

}  // namespace ccmk
