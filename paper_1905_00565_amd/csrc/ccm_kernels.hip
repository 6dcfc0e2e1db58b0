// ccm_kernels.hip -- gfx950 kernels of the simplex cross-map.
//
// The hot path of convergent cross mapping (paper, Section 3.2): for every
// query point of a shadow manifold, the E+1 nearest vectors of a random
// library subsample, found by brute force over all library vectors; then a
// simplex-projection prediction of the other series (Section 2.1) and the
// Pearson skill of the predictions (Section 2.1), for r subsamples per
// library size L (Introduction).
//
// Kernels, in pipeline order:
//   k_ingest       double series -> float series (round to nearest even)
//   k_embed        lagged-coordinate embedding, AoS float[n_e][E]
//   k_sort_chunks  visiting-order keys of each order set (value, or Hilbert
//                  position over a few lag coordinates), sorted in chunks
//   k_merge_runs   the chunks merged
//   k_kd_level     one level of the k-d refinement of the orders
//   k_query_order  each embedding's points in its set's visiting order
//   k_sample       library subsamples: selection sampling driven by SplitMix64
//   k_gather       each library laid out in visiting order, plus the
//                  position every query tile starts scanning from
//   k_crossmap     fused distance / top-(E+1) / prediction / Pearson moments,
//                  one workgroup per (realization, query tile) work item,
//                  optionally persistent with an atomic work queue
//   k_masks, k_order_points, k_rows, k_walk, k_walk_moments
//                  the same result through sorted neighbour rows shared by
//                  all libraries of an embedding (ccm_walk.h), for the
//                  realizations where the planner finds that cheaper
//   k_finalize     merge the per-tile moments of each realization -> rho
//
// Arithmetic that must agree bit for bit with the CPU oracle:
//   d2 = sum_k (q_k - p_k)^2 in binary32 as acc = fma(diff, diff, acc),
//   k ascending from acc = +0 (the first term is the plain product, which is
//   the same value), no other contraction (-ffp-contract=off);
//   neighbours are the first E+1 candidates in (d2, j) order.
// The cross-map kernels themselves are templates in ccm_device.h, compiled
// once per E by ccm_inst.hip; this file holds the kernels that do not depend
// on E and the launchers that dispatch by E.
//
// The order in which candidates are visited is free: selection uses the exact
// (d2, j) key.  Queries are grouped and candidates visited roughly nearest
// first (along a space-filling curve) only so that the running lists settle
// early and the insertion path stays rare; the scan still evaluates every
// (query, candidate) pair.
#include "ccm_walk.h"
#include "ccm_inst.h"
#include "ccm_copy.h"

namespace ccmk {

// ---------------------------------------------------------------------------
// ingest and embedding
// ---------------------------------------------------------------------------

__global__ void k_ingest(const IngestJob* __restrict__ jobs,
                         const double* __restrict__ src,
                         float* __restrict__ dst) {
  const IngestJob J = jobs[blockIdx.y];
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < J.n;
       t += (int64_t)gridDim.x * blockDim.x)
    dst[J.dst_off + t] = __double2float_rn(src[J.src_off + t]);
}

// Backward lags: embedded point i sits at time i + (E-1) tau and its
// coordinate k is the series at that time minus k tau.
__global__ void k_embed(const EmbedJob* __restrict__ jobs,
                        const float* __restrict__ s32,
                        float* __restrict__ emb) {
  const EmbedJob J = jobs[blockIdx.y];
  const int64_t n = J.n_e * J.E;
  const float* __restrict__ s = s32 + J.src_off;
  float* __restrict__ o = emb + J.dst_off;
  for (int64_t x = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; x < n;
       x += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = x / J.E;
    const int k = (int)(x - i * J.E);
    o[x] = s[i + (int64_t)(J.E - 1 - k) * J.tau];
  }
}

// Position of (x, y) on the Hilbert curve filling [0, 2^16)^2 (the classic
// quadrant-by-quadrant construction: at each scale the quadrant contributes
// s*s*((3*rx) ^ ry) and the remaining coordinates are reflected/swapped into
// that quadrant's frame).
__device__ __forceinline__ uint32_t hilbert16(uint32_t x, uint32_t y) {
  uint32_t d = 0;
  for (uint32_t s = 1u << 15; s > 0; s >>= 1) {
    const uint32_t rx = (x & s) ? 1u : 0u;
    const uint32_t ry = (y & s) ? 1u : 0u;
    d += s * s * ((3u * rx) ^ ry);
    if (ry == 0) {
      if (rx == 1) {
        x = 0xffffu - x;
        y = 0xffffu - y;
      }
      const uint32_t t = x;
      x = y;
      y = t;
    }
  }
  return d;
}

// Order-preserving map of binary32 to uint32.
__device__ __forceinline__ uint32_t ordered_bits(float v) {
  const uint32_t b = __float_as_uint(v);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

__device__ __forceinline__ float from_ordered_bits(uint32_t u) {
  return __uint_as_float((u & 0x80000000u) ? u ^ 0x80000000u : ~u);
}

// Index on the n-dimensional Hilbert curve of 32 / n bits per axis (n known to
// the compiler, so that x stays in registers): Skilling's transpose form
// (J. Skilling, "Programming the Hilbert curve", AIP Conf. Proc. 707, 2004) --
// undo the excess work of the recursive reflections and exchanges from the top
// bit down, Gray-encode across axes, then read the index bits axis-interleaved,
// top bit first.
template <int n>
__device__ __forceinline__ uint32_t hilbert_nd(uint32_t (&x)[n]) {
  constexpr int b = 32 / n;
  const uint32_t top = 1u << (b - 1);
  for (uint32_t q = top; q > 1; q >>= 1) {
    const uint32_t low = q - 1;
#pragma unroll
    for (int i = 0; i < n; ++i) {
      if (x[i] & q) {
        x[0] ^= low;
      } else {
        const uint32_t t = (x[0] ^ x[i]) & low;
        x[0] ^= t;
        x[i] ^= t;
      }
    }
  }
#pragma unroll
  for (int i = 1; i < n; ++i) x[i] ^= x[i - 1];
  uint32_t t = 0;
  for (uint32_t q = top; q > 1; q >>= 1)
    if (x[n - 1] & q) t ^= q - 1;
#pragma unroll
  for (int i = 0; i < n; ++i) x[i] ^= t;
  uint32_t h = 0;
  for (int bit = b - 1; bit >= 0; --bit)
#pragma unroll
    for (int i = 0; i < n; ++i) h = (h << 1) | ((x[i] >> bit) & 1u);
  return h;
}

// ---------------------------------------------------------------------------
// library subsamples
// ---------------------------------------------------------------------------

// SplitMix64 output mix (Steele, Lea & Flood, OOPSLA 2014).
__device__ __forceinline__ uint64_t sm_mix(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  return z ^ (z >> 31);
}

// Selection sampling (Knuth, TAOCP Vol. 2, Sec. 3.4.2, Algorithm S): visit
// candidates 0..n_e-1 in order and take candidate j with probability
// (needed / remaining); the uniform integer below (n_e - j) is the high word of
// the 64x64-bit product of one SplitMix64 draw with (n_e - j).  The stream of
// a library is keyed by (seed, E, tau, L_eff, r) folded through the mix.
// Once every remaining candidate is needed the rest are taken without draws:
// the test would accept each of them whatever the draw.
//
// One wavefront per library.  The stream's state advances by the same
// constant for every candidate visited, so candidate j's draw is the output
// mix of (keyed state + (j+1) gamma): the 64 lanes form the draws and their
// integers u_j below (n_e - j) of 64 consecutive candidates at once.  The
// decisions depend on how many were taken before (t_j = needed before j;
// take j when u_j < t_j), but within 64 candidates t_j is at most 63 below
// the step's t_0: u_j < t_0 - 63 is taken and u_j >= t_0 is not whatever
// came before, and only the lanes in between are decided one after another,
// in candidate order, with the count of takes below them.  Then t_j is known
// for every lane, and the first j with t_j = n_e - j (every remaining one
// needed) takes the rest.  Each u_j is below n_e < 2^31.
constexpr uint64_t kGamma = 0x9e3779b97f4a7c15ull;

// The candidates at or below n_e - 1 among the 64 from j0 on.
__device__ __forceinline__ uint64_t tail_word(int64_t ne, int64_t j0) {
  return ne - j0 >= 64 ? ~0ull : ~(~0ull << (ne - j0));
}

template <bool BITS>
__device__ __forceinline__ void sample_members(const SampleJob& J,
                                               int32_t* __restrict__ out_pool,
                                               uint64_t* __restrict__ bit_pool) {
  const int lane = threadIdx.x & 63;
  uint64_t st = 0;
  st = sm_mix(st ^ J.seed);
  st = sm_mix(st ^ (uint64_t)(int64_t)J.E);
  st = sm_mix(st ^ (uint64_t)(int64_t)J.tau);
  st = sm_mix(st ^ (uint64_t)J.l_eff);
  st = sm_mix(st ^ (uint64_t)(int64_t)J.r_index);
  int32_t* __restrict__ out = out_pool + J.out_off;
  const int64_t ne = J.n_e, le = J.l_eff;
  const bool list = !BITS || J.no_list == 0;
  uint64_t* __restrict__ bits = BITS ? bit_pool + (J.bits - 1) : nullptr;
  const int64_t nw = (ne + 63) / 64;
  uint64_t word = 0;                              // word 64 * (j0 / 4096) + lane
  const uint64_t below_lane = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  int64_t s = 0;                                  // taken so far
  int64_t j0 = 0;
  for (; s < le && j0 < ne; j0 += 64) {
    const int64_t j = j0 + lane;
    const bool valid = j < ne;
    int64_t u = 0;
    if (valid)
      u = (int64_t)__umul64hi(sm_mix(st + (uint64_t)(j + 1) * kGamma), (uint64_t)(ne - j));
    const int64_t t0 = le - s;
    uint64_t take = __builtin_amdgcn_ballot_w64(valid && u + 63 < t0);
    uint64_t open = __builtin_amdgcn_ballot_w64(valid && u + 63 >= t0 && u < t0);
    while (open) {                                // in candidate order
      const int l = __builtin_ctzll(open);
      open &= open - 1ull;
      const int64_t tl = t0 - __popcll(take & ((1ull << l) - 1ull));
      const int64_t ul = (int64_t)(uint32_t)__builtin_amdgcn_readlane((int)u, l);
      if (ul < tl) take |= 1ull << l;
    }
    // the first candidate from which every remaining one is needed
    const int64_t tj = t0 - __popcll(take & below_lane);
    const uint64_t full = __builtin_amdgcn_ballot_w64(valid && tj == ne - j);
    int64_t rest = -1;
    if (full) {
      const int l = __builtin_ctzll(full);
      rest = j0 + l;
      take &= (1ull << l) - 1ull;
    }
    if (list && ((take >> lane) & 1ull)) out[s + __popcll(take & below_lane)] = (int32_t)j;
    s += __popcll(take);
    if (rest >= 0) {
      if (list)
        for (int64_t k = lane; k < le - s; k += 64) out[s + k] = (int32_t)(rest + k);
      s = le;
      // candidates rest .. n_e - 1, all of them: to the end of the bitmap
      take |= (~0ull << (rest - j0)) & tail_word(ne, j0);
    }
    if (BITS) {
      const int64_t x = j0 >> 6;
      if (lane == (int)(x & 63)) word = take;
      if ((x & 63) == 63) {
        bits[x - 63 + lane] = word;
        word = 0;
      }
      if (rest >= 0) {
        // the words not yet stored of this 64, then the remaining ones
        const int64_t y0 = (x & ~63ll) + ((x & 63) == 63 ? 64 : 0);
        for (int64_t y = y0 + lane; y < nw; y += 64)
          bits[y] = y <= x ? word : tail_word(ne, y * 64);
        return;
      }
    }
  }
  if (BITS) {
    // every candidate is taken already: the pending words, then zeros
    const int64_t x = j0 >> 6;                    // words formed
    for (int64_t y = (x & ~63ll) + lane; y < nw; y += 64) bits[y] = y < x ? word : 0ull;
  }
}

// One draw: its list, its bitmap, or both.  The loop is one serial chain per
// library, and a draw without a bitmap does not carry the bitmap's steps: with
// them 19.5 ms for 4 x 10^6 candidates, without 16.7.
__device__ __forceinline__ void sample_library(const SampleJob& J,
                                               int32_t* __restrict__ out_pool,
                                               uint64_t* __restrict__ bit_pool) {
  if (J.bits > 0)
    sample_members<true>(J, out_pool, bit_pool);
  else
    sample_members<false>(J, out_pool, bit_pool);
}

__global__ __launch_bounds__(256) void k_sample(const SampleJob* __restrict__ jobs,
                                                int64_t n_jobs, int32_t* __restrict__ out_pool,
                                                uint64_t* __restrict__ bit_pool) {
  const int64_t id = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (id < n_jobs) sample_library(jobs[id], out_pool, bit_pool);
}

// ---------------------------------------------------------------------------
// visiting orders
// ---------------------------------------------------------------------------

// Sum of v over the threads below this one of a workgroup of BLOCK, and the
// sum over all of them.  One barrier: calls in a row take turns at two sets
// of s_sum (turn 0 and 1).
template <int BLOCK>
__device__ __forceinline__ int block_scan(int v, int (*s_sum)[BLOCK / 64], int turn, int& total) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  int inc = v;
#pragma unroll
  for (int s = 1; s < 64; s <<= 1) {
    const int y = __shfl_up(inc, s, 64);
    if (lane >= s) inc += y;
  }
  if (lane == 63) s_sum[turn][wave] = inc;
  __syncthreads();
  int before = inc - v;
  total = 0;
#pragma unroll
  for (int w = 0; w < BLOCK / 64; ++w) {
    if (w < wave) before += s_sum[turn][w];
    total += s_sum[turn][w];
  }
  return before;
}

// Smallest and largest value of the series by a workgroup (every thread gets
// both; s_lo, s_hi: one entry per wavefront).
__device__ __forceinline__ void series_range(const float* __restrict__ s, int64_t n, float* s_lo,
                                             float* s_hi, float& a, float& b) {
  a = __builtin_inff();
  b = -__builtin_inff();
#pragma unroll 4
  for (int64_t t = threadIdx.x; t < n; t += blockDim.x) {
    a = fminf(a, s[t]);
    b = fmaxf(b, s[t]);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    a = fminf(a, __shfl_xor(a, o, 64));
    b = fmaxf(b, __shfl_xor(b, o, 64));
  }
  if ((threadIdx.x & 63) == 0) {
    s_lo[threadIdx.x >> 6] = a;
    s_hi[threadIdx.x >> 6] = b;
  }
  __syncthreads();
  for (int w = 0; w < (int)blockDim.x / 64; ++w) {
    a = fminf(a, s_lo[w]);
    b = fmaxf(b, s_hi[w]);
  }
}

// The ranges of the sets' series, once for sets of several chunks (one
// workgroup per set).
__global__ __launch_bounds__(1024) void k_series_range(const OrderJob* __restrict__ jobs,
                                                       const float* __restrict__ s32,
                                                       float2* __restrict__ range) {
  __shared__ float s_lo[16], s_hi[16];
  const OrderJob J = jobs[blockIdx.x];
  if (J.dims == 1) return;                         // not used
  float a, b;
  series_range(s32 + J.src_off, J.n, s_lo, s_hi, a, b);
  if (threadIdx.x == 0) range[blockIdx.x] = make_float2(a, b);
}

// Keys of the order sets (see OrderJob), sorted in chunks of `chunk` positions
// (a power of two from 64 to kSortChunk): a workgroup forms its chunk's keys in LDS and ranks 64 of them
// against all (by key, then time index: the ranks are all different, the sort
// stable), each wavefront over its share of the chunk.  The (key, time index)
// go to out64 by rank (merged by k_merge_runs), or with one chunk per set the
// indices to out32.  range: the sets' ranges (k_series_range), or null: taken
// here.  Grid ((n / 64) rounded up, sets and slices of draws): the library
// draws of a short call ride along, since neither needs the other (a launch of
// its own: 7 us of a pair of 120 points, 16 of one of 777).
//
// Latency-bound at every size: the 4096^2 comparisons (two instructions each)
// take 1 us over a chip's worth of wavefronts, while a bitonic network in one
// workgroup's LDS has 78 dependent steps.  Two sets of 5003 points: a radix
// sort with one workgroup per set 132 us, bitonic chunks of 4096 and a merge
// 47, here 12 and three merges of 5; two of 10^5: 2.0 ms and 0.09.
constexpr int kSortChunk = 4096;

__global__ __launch_bounds__(1024) void k_sort_chunks(const OrderJob* __restrict__ jobs,
                                                      const float* __restrict__ s32,
                                                      const float2* __restrict__ range,
                                                      int chunk, uint64_t* __restrict__ out64,
                                                      int32_t* __restrict__ out32, int n_sets,
                                                      Draws draws) {
  __shared__ __align__(16) uint32_t key[kSortChunk];
  __shared__ float s_lo[16], s_hi[16];
  __shared__ int s_less[16][64];
  if ((int)blockIdx.y >= n_sets) {                 // a wavefront per draw
    const int64_t id = ((int64_t)(blockIdx.y - n_sets) * gridDim.x + blockIdx.x) *
                           (blockDim.x / 64) +
                       __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (id < draws.n) sample_library(draws.jobs[id], draws.out, draws.bits);
    return;
  }
  const OrderJob J = jobs[blockIdx.y];
  const float* __restrict__ s = s32 + J.src_off;
  const int tid = threadIdx.x;
  const int nt = blockDim.x;
  const int dims = J.dims;
  const int64_t first = (int64_t)blockIdx.x * 64;
  if (first >= J.n) return;                        // the whole workgroup
  const int64_t c0 = first & ~(int64_t)(chunk - 1);
  const int own = (int)(first - c0);
  const int m = (int)min((int64_t)chunk, J.n - c0);
  const int nw = nt / 64;
  const int share = (m + 4 * nw - 1) / (4 * nw) * 4;   // keys per wavefront
  int64_t lag_max = 0;
#pragma unroll
  for (int d = 0; d < 4; ++d)
    if (d < dims) lag_max = max(lag_max, (int64_t)J.lag[d]);
  float lo = 0.f, scale = 0.f, top = 0.f;
  if (dims > 1) {
    float hi;
    if (range) {
      lo = range[blockIdx.y].x;
      hi = range[blockIdx.y].y;
    } else {
      series_range(s, J.n, s_lo, s_hi, lo, hi);
    }
    top = (float)((1u << (dims == 2 ? 16 : 8)) - 1u);
    const float span = hi - lo;
    scale = span > 0.f ? top / span : 0.f;
  }
  for (int x = tid; x < share * nw && x < kSortChunk; x += nt) {
    const int64_t i = c0 + x;
    uint32_t u = 0xffffffffu;                      // past the end: counts nowhere
    if (x < m && i + lag_max < J.n) {
      if (dims == 1) {
        u = ordered_bits(s[i + J.lag[0]]);
      } else {
        // (two coordinates or four: indexed at run time they lived in scratch
        // memory, 80 bytes a lane, which a launch has to find on the device)
        uint32_t g[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int d = 0; d < 4; ++d)
          if (d < dims)
            g[d] = (uint32_t)fminf(top, fmaxf(0.f, (s[i + J.lag[d]] - lo) * scale));
        u = dims == 2 ? hilbert16(g[0], g[1]) : hilbert_nd<4>(g);
      }
    }
    key[x] = u;
  }
  __syncthreads();
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const bool mine = own + lane < m;
  const uint32_t u = mine ? key[own + lane] : 0u;
  int less = 0;
  const int a = min(wave * share, kSortChunk), b = min(a + share, kSortChunk);
  // before the 64 keys equal ones count, after them not
  const uint4* __restrict__ k4 = reinterpret_cast<const uint4*>(key);
#pragma unroll 4
  for (int q = a / 4; q < min(b, own) / 4; ++q) {
    const uint4 v = k4[q];
    less += (v.x <= u ? 1 : 0) + (v.y <= u ? 1 : 0) + (v.z <= u ? 1 : 0) + (v.w <= u ? 1 : 0);
  }
  for (int x = max(a, own); x < min(b, own + 64); ++x)
    less += key[x] < u || (key[x] == u && x < own + lane) ? 1 : 0;
#pragma unroll 4
  for (int q = max(a, own + 64) / 4; q < b / 4; ++q) {
    const uint4 v = k4[q];
    less += (v.x < u ? 1 : 0) + (v.y < u ? 1 : 0) + (v.z < u ? 1 : 0) + (v.w < u ? 1 : 0);
  }
  s_less[wave][lane] = less;
  __syncthreads();
  if (wave == 0 && mine) {
    int r = 0;
    for (int w = 0; w < nw; ++w) r += s_less[w][lane];
    const int64_t i = first + lane;
    if (out64)
      out64[J.key_off + c0 + r] = ((uint64_t)u << 32) | (uint32_t)i;
    else
      out32[J.key_off + c0 + r] = (int32_t)i;
  }
}

// One merge of sorted runs of `run` keys into runs twice as long, every set
// (n keys each) at once: a key's place is its place in its own run plus the
// number of smaller keys in the other one (found by bisection; the keys are
// all different).  The last merge writes the indices only (out32).
__global__ __launch_bounds__(256) void k_merge_runs(const uint64_t* __restrict__ src, int64_t run,
                                                    int64_t n, uint64_t* __restrict__ out64,
                                                    int32_t* __restrict__ out32) {
  const int64_t x = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (x >= n) return;
  const uint64_t* __restrict__ k = src + (int64_t)blockIdx.y * n;
  const uint64_t key = k[x];
  const int64_t r = x / run;
  const int64_t o = (r ^ 1) * run;                 // the other run
  int64_t lo = min(o, n), hi = min(o + run, n);
  const int64_t first = lo;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (k[mid] < key) lo = mid + 1;
    else hi = mid;
  }
  const int64_t at = (int64_t)blockIdx.y * n + (r & ~1ll) * run + (x - r * run) + (lo - first);
  if (out64)
    out64[at] = key;
  else
    out32[at] = (int32_t)(uint32_t)key;
}

// One level of the k-d refinement (see OrderJob): workgroup (x, y) splits
// node x of set y -- positions [lo, hi) = [x n_e / 2^level, (x+1) n_e /
// 2^level) of the set's order -- at its median along the coordinate with the
// widest range over the node (the first such coordinate on ties).  The h =
// mid - lo smallest (coordinate, position) entries go to [lo, mid), the rest
// to [mid, hi), each side in its input order, where mid = (2x+1) n_e /
// 2^(level+1) is the next level's boundary between the node's halves.  The
// h-th smallest coordinate T is found by counting the entries in equal bins
// of the range and ranking those of the bin that holds it, or, with many in
// that bin, by a radix select on the ordered bits (11, 11 and 10 bits); the
// entries below T and the first ones equal to T make up the lower half (the
// node's keys are formed once into `keys`, scratch of the pool's size).  Sets set0 + blockIdx.y.  Input
// `order`, output `out`; nodes that do not split and entries outside the
// nodes are copied.
//
// Latency-bound (a node is one workgroup): every step is parallel over the
// workgroup, and the top levels' nodes get 1024 threads.  With four 8-bit
// passes, each ended by one thread's walk over the counters, and a copy of
// the pool per level, two sets of 777 points took 46 us a level and two of
// 10^5 2.3 ms in all; now 9 us and 0.95 ms.
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_kd_level(const OrderJob* __restrict__ orders, int set0,
                                                    int level, const float* __restrict__ emb,
                                                    const int32_t* __restrict__ order,
                                                    uint32_t* __restrict__ keys,
                                                    int32_t* __restrict__ out) {
  constexpr int kNW = BLOCK / 64;
  constexpr int kBins = 2048;
  constexpr int kPer = kBins / BLOCK;              // counters per thread
  __shared__ float s_lo[kNW][kMaxE], s_hi[kNW][kMaxE];
  __shared__ uint32_t hist[kBins];
  __shared__ uint32_t s_key[BLOCK];
  __shared__ uint32_t s_pick[3];
  __shared__ int s_sum[2][kNW];
  __shared__ int s_n, s_nan;
  const OrderJob J = orders[set0 + (int)blockIdx.y];
  const int tid = threadIdx.x;
  const int64_t x = blockIdx.x;
  const int32_t* __restrict__ o = order + J.key_off;
  int32_t* __restrict__ w = out + J.key_off;
  if (J.kd_E <= 0 || level >= J.kd_levels) {       // no (further) refinement: its share
    const int64_t b = ((x + 1) * J.n) >> level;
    for (int64_t p = ((x * J.n) >> level) + tid; p < b; p += BLOCK) w[p] = o[p];
    return;
  }
  const int E = J.kd_E;
  const int64_t lo = (x * J.kd_n_e) >> level;
  const int64_t hi = ((x + 1) * J.kd_n_e) >> level;
  const int64_t mid = ((2 * x + 1) * J.kd_n_e) >> (level + 1);
  const int64_t h = mid - lo;                       // entries of the lower half
  if (x == 0)                                       // past the embedded points
    for (int64_t p = J.kd_n_e + tid; p < J.n; p += BLOCK) w[p] = o[p];
  if (h <= 0 || h >= hi - lo) {                     // nothing moves
    for (int64_t p = lo + tid; p < hi; p += BLOCK) w[p] = o[p];
    return;
  }
  const float* __restrict__ e = emb + J.kd_emb_off;

  // the widest coordinate: every coordinate's range in one pass
  float mn[kMaxE], mx[kMaxE];
#pragma unroll
  for (int k = 0; k < kMaxE; ++k) {
    mn[k] = __builtin_inff();
    mx[k] = -__builtin_inff();
  }
  for (int64_t p = lo + tid; p < hi; p += BLOCK) {
    const float* __restrict__ v = e + (int64_t)o[p] * E;
#pragma unroll
    for (int k = 0; k < kMaxE; ++k)
      if (k < E) {
        mn[k] = fminf(mn[k], v[k]);
        mx[k] = fmaxf(mx[k], v[k]);
      }
  }
  const int wave = tid >> 6;
#pragma unroll
  for (int k = 0; k < kMaxE; ++k) {
    if (k >= E) break;
#pragma unroll
    for (int sh = 32; sh > 0; sh >>= 1) {
      mn[k] = fminf(mn[k], __shfl_xor(mn[k], sh, 64));
      mx[k] = fmaxf(mx[k], __shfl_xor(mx[k], sh, 64));
    }
    if ((tid & 63) == 0) {
      s_lo[wave][k] = mn[k];
      s_hi[wave][k] = mx[k];
    }
  }
  __syncthreads();
  int d = 0;
  float width = -1.f, least = 0.f;
  for (int k = 0; k < E; ++k) {
    float a = s_lo[0][k], b = s_hi[0][k];
#pragma unroll
    for (int wv = 1; wv < kNW; ++wv) {
      a = fminf(a, s_lo[wv][k]);
      b = fmaxf(b, s_hi[wv][k]);
    }
    if (b - a > width) {
      width = b - a;
      least = a;
      d = k;
    }
  }

  // the keys, counted in 2048 equal bins of the node's range (values map to
  // bins monotonically; without a finite scale all are in bin 0)
  uint32_t* __restrict__ kc = keys + J.key_off;
  const float scale = (float)(kBins - 1) / width;
  const bool binned = width > 0.f && width < __builtin_inff() && scale < __builtin_inff();
  auto bin_of = [&](float v) {
    return binned ? min(kBins - 1, (int)((v - least) * scale)) : 0;
  };
  for (int b = tid; b < kBins; b += BLOCK) hist[b] = 0u;
  if (tid == 0) s_n = s_nan = 0;
  __syncthreads();
  for (int64_t p = lo + tid; p < hi; p += BLOCK) {
    const float v = e[(int64_t)o[p] * E + d];
    if (v != v) s_nan = 1;
    kc[p] = ordered_bits(v);
    atomicAdd(&hist[bin_of(v)], 1u);
  }
  __syncthreads();
  // the counter that holds the entry of rank `rank`, and its rank in there
  auto pick = [&](uint32_t rank, int turn) {
    uint32_t c[kPer], sum = 0;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      c[u] = hist[tid * kPer + u];
      sum += c[u];
    }
    int all;
    uint32_t cum = (uint32_t)block_scan<BLOCK>((int)sum, s_sum, turn, all);
    if (cum <= rank && rank < cum + sum) {          // one thread
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        if (rank >= cum && rank < cum + c[u]) {
          s_pick[0] = (uint32_t)(tid * kPer + u);
          s_pick[1] = rank - cum;
          s_pick[2] = c[u];
        }
        cum += c[u];
      }
    }
    __syncthreads();
  };
  // the key T of rank h - 1 (0-based), and how many entries equal to it are
  // in the lower half
  uint32_t T;
  int eq_left;
  pick((uint32_t)(h - 1), 0);
  if (binned && !s_nan && s_pick[2] <= (uint32_t)BLOCK) {
    // the bin's few entries, each ranked against the others
    const int bin = (int)s_pick[0];
    const int rank = (int)s_pick[1];
    for (int64_t p = lo + tid; p < hi; p += BLOCK) {
      const uint32_t key = kc[p];
      if (bin_of(from_ordered_bits(key)) == bin) s_key[atomicAdd(&s_n, 1)] = key;
    }
    __syncthreads();
    const int n = s_n;
    if (tid < n) {
      const uint32_t key = s_key[tid];
      int less = 0, same = 0;
      for (int x = 0; x < n; ++x) {
        less += s_key[x] < key ? 1 : 0;
        same += s_key[x] == key ? 1 : 0;
      }
      if (less <= rank && rank < less + same) {     // equal keys write the same
        s_pick[0] = key;
        s_pick[1] = (uint32_t)(rank - less);
      }
    }
    __syncthreads();
    T = s_pick[0];
    eq_left = (int)s_pick[1] + 1;
  } else {
    // many in one bin: radix select over the keys
    uint32_t prefix = 0u, mask = 0u;
    uint32_t rank = (uint32_t)(h - 1);
#pragma unroll 1
    for (int pass = 0; pass < 3; ++pass) {
      const int shift = pass == 0 ? 21 : (pass == 1 ? 10 : 0);
      const uint32_t digit = pass == 2 ? 1023u : 2047u;
      for (int b = tid; b < kBins; b += BLOCK) hist[b] = 0u;
      __syncthreads();
      for (int64_t p = lo + tid; p < hi; p += BLOCK) {
        const uint32_t key = kc[p];
        if ((key & mask) == prefix) atomicAdd(&hist[(key >> shift) & digit], 1u);
      }
      __syncthreads();
      pick(rank, (pass & 1) ^ 1);
      prefix |= s_pick[0] << shift;
      mask |= digit << shift;
      rank = s_pick[1];
      __syncthreads();
    }
    T = prefix;
    eq_left = (int)rank + 1;
  }

  // stable partition, four consecutive entries per thread at a time
  constexpr int kRun = 4;
  int64_t at_lo = lo, at_hi = mid;
  int eq_seen = 0;
  for (int64_t base = lo; base < hi; base += BLOCK * kRun) {
    const int64_t p0 = base + (int64_t)tid * kRun;
    uint32_t key[kRun];
    int32_t idx[kRun];
    int n_eq = 0, n_in = 0;
#pragma unroll
    for (int u = 0; u < kRun; ++u) {
      const bool in = p0 + u < hi;
      key[u] = in ? kc[p0 + u] : 0u;
      idx[u] = in ? o[p0 + u] : 0;
      n_in += in ? 1 : 0;
      n_eq += in && key[u] == T ? 1 : 0;
    }
    int all_eq, all_left;
    int eq = eq_seen + block_scan<BLOCK>(n_eq, s_sum, 0, all_eq);
    bool left[kRun];
    int n_left = 0;
#pragma unroll
    for (int u = 0; u < kRun; ++u) {
      const bool in = u < n_in;
      left[u] = in && (key[u] < T || (key[u] == T && eq < eq_left));
      if (in && key[u] == T) ++eq;
      n_left += left[u] ? 1 : 0;
    }
    const int before = block_scan<BLOCK>(n_left, s_sum, 1, all_left);
    int64_t to_lo = at_lo + before;
    int64_t to_hi = at_hi + ((int64_t)tid * kRun - before);
#pragma unroll
    for (int u = 0; u < kRun; ++u) {
      if (u >= n_in) break;
      if (left[u]) w[to_lo++] = idx[u];
      else w[to_hi++] = idx[u];
    }
    const int64_t n_tile = hi - base < BLOCK * kRun ? hi - base : BLOCK * kRun;
    at_lo += all_left;
    at_hi += n_tile - all_left;
    eq_seen += all_eq;
  }
}

// Embedded points in visiting order: the order set restricted to indices
// below n_e.  Workgroup (x, y) places the entries at positions
// [x span, (x+1) span) of embedding y's set, after counting the ones kept before
// them; a k-d set holds exactly the embedded points first.  At most 512 spans:
// the counting reads span * spans^2 / 2 entries (2048 to a span at every length:
// 2.5 s for two sets of 10^8, one workgroup for all 0.24, now 0.026).
__global__ __launch_bounds__(kBlock) void k_query_order(
    const EmbedJob* __restrict__ jobs, int64_t span, const int32_t* __restrict__ order_pool,
    int32_t* __restrict__ qord_pool) {
  __shared__ int s_wave[kBlock / 64];
  const EmbedJob J = jobs[blockIdx.y];
  const int32_t* __restrict__ ord = order_pool + J.order_off;
  int32_t* __restrict__ q = qord_pool + J.qord_off;
  const int64_t a = (int64_t)blockIdx.x * span;
  if (a >= J.n_series) return;                     // the whole workgroup
  const int64_t b = min(a + span, J.n_series);
  if (J.whole || J.n_e == J.n_series) {
    for (int64_t k = a + threadIdx.x; k < min(b, J.n_e); k += kBlock) q[k] = ord[k];
    return;
  }
  int mine = 0;
#pragma unroll 8
  for (int64_t k = threadIdx.x; k < a; k += kBlock) mine += ord[k] < J.n_e ? 1 : 0;
#pragma unroll
  for (int s = 32; s > 0; s >>= 1) mine += __shfl_xor(mine, s, 64);
  if ((threadIdx.x & 63) == 0) s_wave[threadIdx.x >> 6] = mine;
  __syncthreads();
  int64_t out = 0;
#pragma unroll
  for (int w = 0; w < kBlock / 64; ++w) out += s_wave[w];
  __syncthreads();
  for (int64_t base = a; base < b; base += kBlock) {
    const int64_t k = base + threadIdx.x;
    const int64_t i = k < b ? ord[k] : J.n_e;
    const bool f = i < J.n_e;
    int total;
    const int r = block_rank(f, s_wave, total);
    if (f) q[out + r] = (int32_t)i;
    out += total;
  }
}

// Membership words of the libraries of walk groups: bit l of word j is set
// when library l of the group holds embedded point j -- the transpose of the
// libraries' bitmaps, 64 x 64 bits at a time, one library per lane.  Each
// wavefront takes kMaskWords consecutive bitmap words (a cache line of each
// library's).
constexpr int kMaskWords = 8;

__global__ __launch_bounds__(kBlock) void k_masks(const MaskJob* __restrict__ jobs,
                                                  const WalkLib* __restrict__ libs,
                                                  const uint64_t* __restrict__ bit_pool,
                                                  uint64_t* __restrict__ mask_pool) {
  const MaskJob J = jobs[blockIdx.y];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int x0 = ((int)blockIdx.x * kWaves + wave) * kMaskWords;
  const int nw = (J.n_e + 63) / 64;
  const bool mine = lane < J.n_lib;
  const uint64_t* __restrict__ bits = bit_pool + libs[J.lib_first + (mine ? lane : 0)].bit_off;
  const BitTranspose transpose(lane);
  uint64_t v[kMaskWords];
#pragma unroll
  for (int u = 0; u < kMaskWords; ++u) v[u] = mine && x0 + u < nw ? bits[x0 + u] : 0ull;
#pragma unroll
  for (int u = 0; u < kMaskWords; ++u) {
    const uint64_t m = transpose(v[u]);
    const int j = (x0 + u) * 64 + lane;
    if (j < J.n_e) mask_pool[J.mask_off + j] = m;
  }
}

// Nested libraries (an option of this library): the first n_out points of
// the forward Fisher-Yates shuffle (Durstenfeld 1964; Knuth's Algorithm P,
// TAOCP Vol. 2, Sec. 3.4.2) of 0..n_e-1: step k swaps position k with
// position j_k = k + floor(z_k (n_e - k) / 2^64), z_k the k-th SplitMix64
// output of the stream keyed by (seed, E, tau, r).  The first n_list points
// are written out; a job with `bits` also leaves the bitmaps of its libraries
// of segments seg0 .. n_seg - 1 (cumulative, (n_e + 63) / 64 words each).
//
// One workgroup per job; its first wavefront takes 64 steps at a time.  Step
// i touches positions k_i and j_i >= k_i, so it must wait for the steps i' <
// i with j_i' equal to either, and for no other: each lane collects those
// steps in a mask, and runs of steps free of each other swap at once.  With
// the positions in LDS (CAP of them) a run costs a few hundred cycles and
// 64 steps of 10^4 points take one or two; one lane in global memory took
// 0.29 us a step (2.9 ms for 10^4 points, here 0.33).
template <int CAP>
__global__ __launch_bounds__(kBlock) void k_sample_nested(const NestedJob* __restrict__ jobs,
                                                          const int32_t* __restrict__ seg_pool,
                                                          int32_t* __restrict__ scratch,
                                                          int32_t* __restrict__ out_pool,
                                                          uint64_t* __restrict__ bit_pool) {
  constexpr bool kLds = CAP > 0;
  __shared__ uint16_t pos[kLds ? CAP : 1];
  __shared__ uint32_t bm[kLds ? CAP / 32 : 2];
  const NestedJob J = jobs[blockIdx.x];
  int32_t* __restrict__ far = scratch + J.scratch_off;   // CAP == 0
  const int ne = (int)J.n_e;
  const int n_out = (int)J.n_out;
  for (int i = threadIdx.x; i < ne; i += kBlock) {
    if constexpr (kLds) pos[i] = (uint16_t)i;
    else far[i] = i;
  }
  __syncthreads();
  if (threadIdx.x < 64) {
    const int lane = threadIdx.x;
    uint64_t st = 0;
    st = sm_mix(st ^ J.seed);
    st = sm_mix(st ^ (uint64_t)(int64_t)J.E);
    st = sm_mix(st ^ (uint64_t)(int64_t)J.tau);
    st = sm_mix(st ^ (uint64_t)(int64_t)J.r_index);
    for (int k0 = 0; k0 < n_out; k0 += 64) {
      const int k = k0 + lane;
      const bool valid = k < n_out;
      const uint64_t z = sm_mix(st + (uint64_t)(k + 1) * kGamma);
      const int j = valid ? k + (int)__umul64hi(z, (uint64_t)(ne - k)) : -1 - lane;
      uint64_t wait = 0;                            // earlier steps this one waits for
#pragma unroll
      for (int s = 0; s < 63; ++s) {
        const int js = __builtin_amdgcn_readlane(j, s);
        if ((js == k || js == j) && lane > s) wait |= 1ull << s;
      }
      const int n = min(64, n_out - k0);
      for (int s = 0; s < n;) {
        const uint64_t held =
            __builtin_amdgcn_ballot_w64(lane > s && (wait & (~0ull << s)) != 0);
        const int e = held ? min(n, (int)__builtin_ctzll(held)) : n;
        if (lane >= s && lane < e) {
          if constexpr (kLds) {
            const uint16_t a = pos[k], b = pos[j];
            pos[j] = a;
            pos[k] = b;
          } else {
            const int32_t a = far[k], b = far[j];
            far[j] = a;
            far[k] = b;
          }
        }
        __threadfence_block();
        s = e;
      }
    }
  }
  __syncthreads();
  int32_t* __restrict__ out = out_pool + J.out_off;
  for (int i = threadIdx.x; i < (int)J.n_list; i += kBlock) out[i] = kLds ? (int32_t)pos[kLds ? i : 0] : far[i];
  if constexpr (kLds) {
    if (J.bits == 0) return;
    const int32_t* __restrict__ seg = seg_pool + J.seg_off;
    const int nw = (ne + 63) / 64;
    uint64_t* __restrict__ bits = bit_pool + (J.bits - 1);
    for (int w = threadIdx.x; w < 2 * nw; w += kBlock) bm[w] = 0u;
    __syncthreads();
    int done = 0;
    for (int s = J.seg0; s < J.n_seg; ++s) {
      const int end = seg[s + 1];
      for (int i = done + (int)threadIdx.x; i < end; i += kBlock) {
        const uint32_t j = pos[i];
        atomicOr(&bm[j >> 5], 1u << (j & 31u));
      }
      done = end;
      __syncthreads();
      for (int w = threadIdx.x; w < nw; w += kBlock)
        bits[(int64_t)(s - J.seg0) * nw + w] = ((uint64_t)bm[2 * w + 1] << 32) | bm[2 * w];
      __syncthreads();
    }
  }
}

// The library of one realization, laid out contiguously in visiting order
// (coordinates AoS and embedded indices), so the scan
// streams it through the scalar cache with no dependent index load.  For each
// wavefront of each query tile (a wavefront takes a run of consecutive
// queries in the same order) it records the library position of the run's
// middle query: that wavefront's scan starts there and works outward.  One
// workgroup per job; the library's membership bitmask lives in LDS (dynamic
// size).  Jobs marked unsorted keep ascending index order and start every
// scan at position 0.
__global__ __launch_bounds__(kBlock) void k_gather(
    const GatherJob* __restrict__ jobs, const float* __restrict__ emb_pool,
    const int32_t* __restrict__ lib_pool, const int32_t* __restrict__ order_pool,
    float* __restrict__ pts_pool, int32_t* __restrict__ pj_pool,
    int32_t* __restrict__ start_pool) {
  extern __shared__ uint32_t bits[];
  __shared__ int s_wave[2][kBlock / 64];
  const GatherJob J = jobs[blockIdx.x];
  const float* __restrict__ emb = emb_pool + J.emb_off;
  const int32_t* __restrict__ lib = lib_pool + J.lib_off;
  float* __restrict__ pts = pts_pool + J.pts_off;
  int32_t* __restrict__ pj = pj_pool + J.pj_off;
  int32_t* __restrict__ start = start_pool + J.start_off;
  const int E = J.E;
  const int tid = threadIdx.x;

  if (!J.sorted) {
    for (int64_t x = tid; x < J.l_eff * E; x += kBlock) {
      const int64_t c = x / E;
      const int k = (int)(x - c * E);
      pts[x] = emb[(int64_t)lib[c] * E + k];
    }
    for (int64_t c = tid; c < J.l_eff; c += kBlock) pj[c] = lib[c];
    if (J.query_set == 0) {
      const int64_t n_start = (J.n_e + J.qt - 1) / J.qt * kWaves;
      for (int64_t t = tid; t < n_start; t += kBlock) start[t] = 0;
    }
    return;
  }

  const int64_t nw = (J.n_e + 31) / 32;
  for (int64_t w = tid; w < nw; w += kBlock) bits[w] = 0u;
  __syncthreads();
  for (int64_t c = tid; c < J.l_eff; c += kBlock) {
    const int32_t j = lib[c];
    atomicOr(&bits[j >> 5], 1u << (j & 31));
  }
  __syncthreads();

  const int32_t* __restrict__ ord = order_pool + J.order_off;
  int64_t pf = 0;   // embedded points passed so far (in order)
  int64_t pl = 0;   // library points passed so far (in order)
  for (int64_t base = 0; base < J.n_series; base += kBlock) {
    const int64_t k = base + tid;
    const int64_t t = k < J.n_series ? ord[k] : J.n_e;
    const bool fo = t < J.n_e;
    const int64_t i = fo ? t : 0;
    const bool fl = fo && ((bits[i >> 5] >> (i & 31)) & 1u);
    int tot_o, tot_l;
    const int ro = block_rank(fo, s_wave[0], tot_o);
    const int rl = block_rank(fl, s_wave[1], tot_l);
    if (fl) {
      const int64_t c = pl + rl;
      pj[c] = (int32_t)i;
      for (int kk = 0; kk < E; ++kk) pts[c * E + kk] = emb[i * E + kk];
    }
    if (fo && J.query_set == 0) {
      // wavefront w of tile t takes query positions [s*sub, (s+1)*sub) with
      // s = t*kWaves + w; its scan starts at its middle query
      const int64_t sub = J.qt / kWaves;
      const int64_t p = pf + ro;
      const int64_t sw = p / sub;
      const int64_t anchor = min(sw * sub + sub / 2, J.n_e - 1);
      if (p == anchor) start[sw] = (int32_t)(pl + rl);
    }
    pf += tot_o;
    pl += tot_l;
  }
}

__global__ void k_finalize_multi(const Realization* __restrict__ rzs,
                                 const int32_t* __restrict__ self_of, int64_t n_rz,
                                 int m_series, const Sums* __restrict__ partial,
                                 int64_t out_stride_b, double* __restrict__ out) {
  const int64_t x = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (x >= n_rz * m_series) return;
  const int64_t r = x / m_series;
  const int bt = (int)(x - r * m_series);
  const Realization R = rzs[r];
  double rho = __builtin_nan("");
  if (bt != self_of[r]) {
    Sums a;
#pragma unroll
    for (int i = 0; i < 6; ++i) a.v[i] = 0.0;
    a.v[6] = a.v[8] = __builtin_inf();
    a.v[7] = a.v[9] = -__builtin_inf();
    for (int t = 0; t < R.n_tiles; ++t) sums_merge(a, partial[(R.slot_base + t) * m_series + bt]);
    const double n = a.v[0];
    const double vo = n * a.v[3] - a.v[1] * a.v[1];
    const double vp = n * a.v[4] - a.v[2] * a.v[2];
    const double cv = n * a.v[5] - a.v[1] * a.v[2];
    if (a.v[6] < a.v[7] && a.v[8] < a.v[9] && vo > 0.0 && vp > 0.0) rho = cv / sqrt(vo * vp);
  }
  out[R.out_index + bt * out_stride_b] = rho;
}

__global__ void k_zero_int(int* p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

// rho = cov / sqrt(var_t var_p) from the merged moments; NaN when either
// side is constant.
__global__ void k_finalize(const Realization* __restrict__ rzs, int64_t n_rz,
                           const Moments* __restrict__ partial,
                           double* __restrict__ out) {
  const int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (r >= n_rz) return;
  const Realization R = rzs[r];
  Moments a = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  for (int t = 0; t < R.n_tiles; ++t) a = mom_merge(a, partial[R.slot_base + t]);
  double rho = __builtin_nan("");
  if (a.m2t > 0.0 && a.m2p > 0.0) rho = a.c / sqrt(a.m2t * a.m2p);
  out[R.out_index] = rho;
}


// ---------------------------------------------------------------------------
// host-side launchers (the runtime calls only these)
// ---------------------------------------------------------------------------

static inline unsigned blocks_for(int64_t n, int per) {
  int64_t b = (n + per - 1) / per;
  if (b < 1) b = 1;
  if (b > 65535) b = 65535;
  return (unsigned)b;
}

int shared_queries_per_lane(int emax) {
  return emax >= 1 && emax <= kMaxE ? kSharedQ[emax] : 0;
}

int crossmap_queries_per_lane(int E) { return E >= 1 && E <= kMaxE ? kTuneQ[E] : 0; }

hipError_t launch_ingest(const IngestJob* jobs, int n_jobs, int64_t max_n,
                         const double* src, float* dst, hipStream_t st) {
  if (n_jobs <= 0) return hipSuccess;
  k_ingest<<<dim3(blocks_for(max_n, 256), n_jobs), 256, 0, st>>>(jobs, src, dst);
  return hipGetLastError();
}

hipError_t launch_embed(const EmbedJob* jobs, int n_jobs, int64_t max_n,
                        const float* s32, float* emb, hipStream_t st) {
  if (n_jobs <= 0) return hipSuccess;
  k_embed<<<dim3(blocks_for(max_n, 256), n_jobs), 256, 0, st>>>(jobs, s32, emb);
  return hipGetLastError();
}

hipError_t build_orders(const OrderJob* orders, int32_t n_sets, int levels, int64_t n_series,
                        const float* s32, const float* emb, void* mem, hipStream_t st,
                        const Draws& draws) {
  if (n_sets <= 0) return draws.n > 0 ? hipErrorInvalidValue : hipSuccess;
  const int64_t n = n_series * n_sets;
  uint64_t* half[2] = {static_cast<uint64_t*>(mem), static_cast<uint64_t*>(mem) + n};
  int32_t* order = order_of(mem, n);
  int32_t* alt = order + n;
  uint32_t* keys = static_cast<uint32_t*>(mem);    // the first half, free after the sort
  // each level moves the entries to the other array; the last one leaves them
  // in `order`
  int32_t* cur = levels & 1 ? alt : order;
  // every 64 keys form and compare a chunk's: long series in short chunks
  const int chunk = n_series > kSortChunk ? 1024 : kSortChunk;
  const unsigned chunks = (unsigned)((n_series + chunk - 1) / chunk);
  int merges = 0;
  while ((1u << merges) < chunks) ++merges;
  const unsigned blocks = (unsigned)((n_series + 63) / 64);
  // sixteen wavefronts share the chunk's 4096 keys while the chip has room
  const bool few = (int64_t)blocks * n_sets <= 512;
  const unsigned threads = few && std::min<int64_t>(n_series, chunk) > 1024 ? 1024 : 256;
  // the last merge reads the first half and writes into the second
  int at = merges > 0 ? (merges - 1) & 1 : 0;
  for (int32_t s0 = 0; s0 < n_sets; s0 += 65535) {
    const unsigned ny = (unsigned)std::min<int32_t>(65535, n_sets - s0);
    float2* const range = merges > 0 ? reinterpret_cast<float2*>(half[at ^ 1]) + s0 : nullptr;
    if (range) k_series_range<<<ny, 1024, 0, st>>>(orders + s0, s32, range);
    Draws d = s0 == 0 ? draws : Draws{};
    const int64_t per = (int64_t)blocks * (threads / 64);
    const int64_t slices = (d.n + per - 1) / per;
    const bool ride = slices > 0 && ny + slices <= 65535;
    if (slices > 0 && !ride) {
      const hipError_t e = launch_sample(d.jobs, d.n, d.out, d.bits, st);
      if (e != hipSuccess) return e;
    }
    if (!ride) d = Draws{};
    k_sort_chunks<<<dim3(blocks, ny + (ride ? (unsigned)slices : 0u)), threads, 0, st>>>(
        orders + s0, s32, range, chunk, merges > 0 ? half[at] : nullptr, cur, (int)ny, d);
  }
  for (int m = 0; m < merges; ++m) {
    const bool last = m + 1 == merges;
    for (int32_t s0 = 0; s0 < n_sets; s0 += 65535) {
      const unsigned ny = (unsigned)std::min<int32_t>(65535, n_sets - s0);
      const int64_t off = (int64_t)s0 * n_series;
      k_merge_runs<<<dim3((unsigned)((n_series + 255) / 256), ny), 256, 0, st>>>(
          half[at] + off, (int64_t)chunk << m, n_series,
          last ? nullptr : half[at ^ 1] + off, cur + off);
    }
    at ^= 1;
  }
  for (int lv = 0; lv < levels; ++lv) {
    int32_t* nxt = cur == order ? alt : order;
    for (int32_t s0 = 0; s0 < n_sets; s0 += 65535) {
      const unsigned ny = (unsigned)std::min<int32_t>(65535, n_sets - s0);
      const dim3 grid(1u << lv, ny);
      if ((n_series >> lv) > 2048)
        k_kd_level<1024><<<grid, 1024, 0, st>>>(orders, s0, lv, emb, cur, keys, nxt);
      else
        k_kd_level<256><<<grid, 256, 0, st>>>(orders, s0, lv, emb, cur, keys, nxt);
    }
    cur = nxt;
  }
  return hipGetLastError();
}

hipError_t launch_query_order(const EmbedJob* jobs, int n_jobs, int64_t n_series,
                              const int32_t* order, int32_t* qord, hipStream_t st) {
  if (n_jobs <= 0) return hipSuccess;
  const int64_t span = query_order_span(n_series);
  const unsigned spans = (unsigned)((n_series + span - 1) / span);
  for (int j0 = 0; j0 < n_jobs; j0 += 65535)
    k_query_order<<<dim3(spans, (unsigned)std::min(65535, n_jobs - j0)), kBlock, 0, st>>>(
        jobs + j0, span, order, qord);
  return hipGetLastError();
}

hipError_t launch_sample(const SampleJob* jobs, int64_t n_jobs, int32_t* out, uint64_t* bits,
                         hipStream_t st) {
  if (n_jobs <= 0) return hipSuccess;
  const unsigned blocks = (unsigned)((n_jobs + 3) / 4);   // one wavefront per library
  k_sample<<<blocks, 256, 0, st>>>(jobs, n_jobs, out, bits);
  return hipGetLastError();
}

// Membership bitmasks up to 48 KiB of LDS per workgroup.
static constexpr int64_t kGatherBitmaskWords = 12 * 1024;

int64_t gather_max_sorted_n_e() { return kGatherBitmaskWords * 32; }

hipError_t launch_gather(const GatherJob* jobs, int64_t n_jobs, int64_t max_n_e,
                         const float* emb, const int32_t* lib, const int32_t* order,
                         float* pts, int32_t* pj, int32_t* start, hipStream_t st) {
  if (n_jobs <= 0) return hipSuccess;
  // max_n_e covers the jobs marked sorted; larger ones must be unsorted
  int64_t words = (max_n_e + 31) / 32;
  if (words > kGatherBitmaskWords) return hipErrorInvalidValue;
  if (words < 1) words = 1;
  k_gather<<<(unsigned)n_jobs, kBlock, (size_t)words * 4, st>>>(jobs, emb, lib, order,
                                                                 pts, pj, start);
  return hipGetLastError();
}

hipError_t launch_masks(const MaskJob* jobs, int n_jobs, int max_ne, const WalkLib* libs,
                        const uint64_t* bits, uint64_t* masks, hipStream_t st) {
  if (n_jobs <= 0 || max_ne <= 0) return hipSuccess;
  constexpr int span = kWaves * kMaskWords * 64;
  const dim3 grid((unsigned)((max_ne + span - 1) / span), (unsigned)n_jobs);
  k_masks<<<grid, kBlock, 0, st>>>(jobs, libs, bits, masks);
  return hipGetLastError();
}

#define CCM_BY_E(E, CALL)                                                             \
  switch (E) {                                                                        \
    case 1: return CALL(1);                                                           \
    case 2: return CALL(2);                                                           \
    case 3: return CALL(3);                                                           \
    case 4: return CALL(4);                                                           \
    case 5: return CALL(5);                                                           \
    case 6: return CALL(6);                                                           \
    case 7: return CALL(7);                                                           \
    case 8: return CALL(8);                                                           \
    case 9: return CALL(9);                                                           \
    case 10: return CALL(10);                                                         \
    default: return hipErrorInvalidValue;                                             \
  }

hipError_t launch_order_points(int E, const RowJob* jobs, int n_jobs, int max_ne,
                               const float* emb, const int32_t* qord, float* pts, float* box,
                               int* todo_n, hipStream_t st) {
  if (n_jobs <= 0 || max_ne <= 0) return hipSuccess;
#define CCM_CALL(e) launch_order_points_e<e>(jobs, n_jobs, max_ne, emb, qord, pts, box, todo_n, st)
  CCM_BY_E(E, CCM_CALL)
#undef CCM_CALL
}

hipError_t launch_rows(int E, const RowJob* jobs, int n_jobs, int max_ne, int max_w,
                       int per_block, const float* pts, const float* box, const int32_t* qord,
                       uint64_t* rows, RowTodo* todo, int* todo_n, hipStream_t st) {
  if (n_jobs <= 0 || max_ne <= 0) return hipSuccess;
  if (max_w < 64 || max_w > kRowMaxW || max_w % 64 != 0 || per_block < 1)
    return hipErrorInvalidValue;
#define CCM_CALL(e) \
  launch_rows_e<e>(jobs, n_jobs, max_ne, max_w, per_block, pts, box, qord, rows, todo, \
                   todo_n, st)
  CCM_BY_E(E, CCM_CALL)
#undef CCM_CALL
}

hipError_t launch_walk(int E, int keys, const WalkGroup* groups,
                       const RowJob* embs, const Item* items, int n_items, int per,
                       const uint64_t* masks, const uint64_t* rows, const int32_t* qord,
                       const float* emb, const double* tgt, double* out, int excl,
                       int query_set, hipStream_t st) {
  if (n_items <= 0) return hipSuccess;
#define CCM_CALL(e)                                                                        \
  launch_walk_e<e>(keys, groups, embs, items, n_items, per, masks, rows, qord, emb, \
                   tgt, out, excl, query_set, st)
  CCM_BY_E(E, CCM_CALL)
#undef CCM_CALL
}

hipError_t launch_spread(int E, int mode, const Realization* rzs, const Item* items, int n_items,
                           const float* emb, const float* pts, const int32_t* pj,
                           const int32_t* qord, const int32_t* start, const double* tgt,
                           double* pred, Moments* partial, int query_set, int window,
                           hipStream_t st) {
  if (n_items <= 0) return hipSuccess;
#define CCM_CALL(e)                                                                       \
  launch_spread_e<e>(mode, rzs, items, n_items, emb, pts, pj, qord, start, tgt, pred, partial, \
                     query_set, window, st)
  CCM_BY_E(E, CCM_CALL)
#undef CCM_CALL
}

hipError_t launch_walk_moments(int E, int shared, const Realization* rzs, const WalkOut* where,
                               const Item* items, int n_items, const double* out,
                               const int32_t* pj, const int32_t* qord, const double* tgt,
                               Moments* partial, int query_set, hipStream_t st) {
  if (n_items <= 0) return hipSuccess;
#define CCM_CALL(e)                                                                       \
  launch_walk_moments_e<e>(shared, rzs, where, items, n_items, out, pj, qord, tgt, partial,     \
                           query_set, st)
  CCM_BY_E(E, CCM_CALL)
#undef CCM_CALL
}

hipError_t launch_multi_keys(int E, const Realization* rzs, const int32_t* self_of,
                             const WalkOut* where, const Item* items, int n_items,
                             const double* keys, const int32_t* pj, const int32_t* qord,
                             const double* tt, int m_series, void* partial, int query_set,
                             hipStream_t st) {
  if (n_items <= 0) return hipSuccess;
#define CCM_CALL(e)                                                                        \
  launch_multi_keys_e<e>(rzs, self_of, where, items, n_items, keys, pj, qord, tt,        \
                         m_series, partial, query_set, st)
  CCM_BY_E(E, CCM_CALL)
#undef CCM_CALL
}

hipError_t launch_multi_group(int E, const Realization* rzs, const int32_t* self_of,
                              const WalkGroup* groups, const WalkLib* libs, const Item* items,
                              int n_items, const double* keys, const int32_t* qord,
                              const double* tt, int m_series, void* partial, hipStream_t st) {
  if (n_items <= 0) return hipSuccess;
#define CCM_CALL(e)                                                                       \
  launch_multi_group_e<e>(rzs, self_of, groups, libs, items, n_items, keys, qord, tt,     \
                          m_series, partial, st)
  CCM_BY_E(E, CCM_CALL)
#undef CCM_CALL
}

hipError_t launch_zero_int(int* p, int n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  k_zero_int<<<(n + 255) / 256, 256, 0, st>>>(p, n);
  return hipGetLastError();
}

hipError_t launch_table_build(int E, const TableJob* jobs, int n_jobs, int max_n_e,
                              const float* emb, int32_t* table, hipStream_t st) {
  if (n_jobs <= 0 || max_n_e <= 0) return hipSuccess;
  switch (E) {
#define CCM_TCASE(e) \
  case e:            \
    return launch_table_build_e<e>(jobs, n_jobs, max_n_e, emb, table, st);
    CCM_TCASE(1) CCM_TCASE(2) CCM_TCASE(3) CCM_TCASE(4) CCM_TCASE(5)
    CCM_TCASE(6) CCM_TCASE(7) CCM_TCASE(8) CCM_TCASE(9) CCM_TCASE(10)
#undef CCM_TCASE
    default:
      return hipErrorInvalidValue;
  }
}

// Two device arrays of n doubles to one buffer, or one buffer to two
// arrays, in a single launch (the device forms' series in and results out).
__global__ void k_copy_pair(const double* __restrict__ a, const double* __restrict__ b,
                            int64_t n, double* __restrict__ dst) {
  for (int64_t x = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; x < 2 * n;
       x += (int64_t)gridDim.x * blockDim.x)
    dst[x] = x < n ? a[x] : b[x - n];
}

__global__ void k_split_pair(const double* __restrict__ src, int64_t n, double* __restrict__ a,
                             double* __restrict__ b) {
  for (int64_t x = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; x < 2 * n;
       x += (int64_t)gridDim.x * blockDim.x) {
    if (x < n)
      a[x] = src[x];
    else
      b[x - n] = src[x];
  }
}

hipError_t launch_copy_pair(const double* a, const double* b, int64_t n, double* dst,
                            hipStream_t st) {
  if (n <= 0) return hipSuccess;
  k_copy_pair<<<blocks_for(2 * n, 256), 256, 0, st>>>(a, b, n, dst);
  return hipGetLastError();
}

hipError_t launch_split_pair(const double* src, int64_t n, double* a, double* b,
                             hipStream_t st) {
  if (n <= 0) return hipSuccess;
  k_split_pair<<<blocks_for(2 * n, 256), 256, 0, st>>>(src, n, a, b);
  return hipGetLastError();
}

hipError_t launch_sample_nested(const NestedJob* jobs, int64_t n_jobs, int64_t max_n_e,
                                const int32_t* seg, int32_t* scratch, int32_t* out_pool,
                                uint64_t* bits, hipStream_t st) {
  if (n_jobs <= 0) return hipSuccess;
  // 34 KB of LDS: four workgroups per CU; 136 KB: one
  if (max_n_e <= 16384)
    k_sample_nested<16384><<<(unsigned)n_jobs, kBlock, 0, st>>>(jobs, seg, scratch, out_pool,
                                                                bits);
  else if (max_n_e <= kNestedLdsNe)
    k_sample_nested<kNestedLdsNe><<<(unsigned)n_jobs, kBlock, 0, st>>>(jobs, seg, scratch,
                                                                       out_pool, bits);
  else
    k_sample_nested<0><<<(unsigned)n_jobs, kBlock, 0, st>>>(jobs, seg, scratch, out_pool, bits);
  return hipGetLastError();
}

hipError_t launch_crossmap_nested(int E, int mode, int grid, const Realization* rzs,
                                  const Item* items, int n_items, int* next,
                                  const float* emb, const float* pts, const int32_t* pj,
                                  const int32_t* qord, const int32_t* start, const double* tgt,
                                  const int32_t* seg, Moments* partial, int window,
                                  hipStream_t st) {
  if (n_items <= 0) return hipSuccess;
  switch (E) {
#define CCM_NCASE(e)                                                                   \
  case e:                                                                              \
    return launch_nested_e<e>(mode, grid, rzs, items, n_items, next, emb, pts, pj, qord, \
                              start, tgt, seg, partial, window, st);
    CCM_NCASE(1) CCM_NCASE(2) CCM_NCASE(3) CCM_NCASE(4) CCM_NCASE(5)
    CCM_NCASE(6) CCM_NCASE(7) CCM_NCASE(8) CCM_NCASE(9) CCM_NCASE(10)
#undef CCM_NCASE
    default:
      return hipErrorInvalidValue;
  }
}

hipError_t launch_crossmap_shared(int emax, int mode, int grid, const Realization* rzs,
                                  const Item* items, int n_items, int* next,
                                  const float* emb, const float* pts, const int32_t* pj,
                                  const int32_t* qord, const int32_t* start, const double* tgt,
                                  Moments* partial, int window, hipStream_t st) {
  if (n_items <= 0) return hipSuccess;
  switch (emax) {
#define CCM_SCASE(e)                                                                     \
  case e:                                                                                \
    return launch_shared_e<e>(mode, grid, rzs, items, n_items, next, emb, pts, pj, qord,  \
                              start, tgt, partial, window, st);
    CCM_SCASE(1) CCM_SCASE(2) CCM_SCASE(3) CCM_SCASE(4) CCM_SCASE(5)
    CCM_SCASE(6) CCM_SCASE(7) CCM_SCASE(8) CCM_SCASE(9) CCM_SCASE(10)
#undef CCM_SCASE
    default:
      return hipErrorInvalidValue;
  }
}

hipError_t launch_crossmap(int E, int mode, int grid,
                           const Realization* rzs, const Item* items,
                           int n_items, int* next, const float* emb,
                           const float* pts, const int32_t* pj,
                           const int32_t* qord, const int32_t* start,
                           const double* tgt, Moments* partial, int query_set,
                           int window, Dump d, const int32_t* table, int table_n_e,
                           hipStream_t st) {
  if (n_items <= 0) return hipSuccess;
  switch (E) {
#define CCM_CASE(e)                                                                         \
  case e:                                                                                   \
    return launch_crossmap_e<e>(mode, grid, rzs, items, n_items, next, emb, pts, pj, qord,  \
                                start, tgt, partial, query_set, window, d, table, table_n_e, \
                                st);
    CCM_CASE(1) CCM_CASE(2) CCM_CASE(3) CCM_CASE(4) CCM_CASE(5)
    CCM_CASE(6) CCM_CASE(7) CCM_CASE(8) CCM_CASE(9) CCM_CASE(10)
#undef CCM_CASE
    default:
      return hipErrorInvalidValue;
  }
}

__global__ void k_transpose_targets(const double* __restrict__ s64, int m, int mp, int64_t n,
                                    double* __restrict__ tt) {
  for (int64_t x = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; x < n * mp;
       x += (int64_t)gridDim.x * blockDim.x) {
    const int64_t t = x / mp;
    const int b = (int)(x - t * mp);
    tt[x] = b < m ? s64[(int64_t)b * n + t] : 0.0;
  }
}

hipError_t launch_transpose_targets(const double* s64, int m_series, int64_t n, double* tt,
                                    hipStream_t st) {
  const int mp = target_stride(m_series);
  k_transpose_targets<<<blocks_for(n * mp, 256), 256, 0, st>>>(s64, m_series, mp, n, tt);
  return hipGetLastError();
}

hipError_t launch_crossmap_multi(int E, int mode, int grid, const Realization* rzs,
                                 const int32_t* self_of, const Item* items, int n_items,
                                 int* next, const float* emb, const float* pts,
                                 const int32_t* pj, const int32_t* qord, const int32_t* start,
                                 const double* tt, int m_series,
                                 void* partial, int query_set, int window,
                                 const int32_t* table, int table_n_e, hipStream_t st) {
  if (n_items <= 0) return hipSuccess;
  switch (E) {
#define CCM_MCASE(e)                                                                      \
  case e:                                                                                 \
    return launch_multi_e<e>(mode, grid, rzs, self_of, items, n_items, next, emb, pts, pj, \
                             qord, start, tt, m_series, partial, query_set, window, table,  \
                             table_n_e, st);
    CCM_MCASE(1) CCM_MCASE(2) CCM_MCASE(3) CCM_MCASE(4) CCM_MCASE(5)
    CCM_MCASE(6) CCM_MCASE(7) CCM_MCASE(8) CCM_MCASE(9) CCM_MCASE(10)
#undef CCM_MCASE
    default:
      return hipErrorInvalidValue;
  }
}

hipError_t launch_finalize_multi(const Realization* rzs, const int32_t* self_of,
                                 int64_t n_rz, int m_series, const void* partial,
                                 int64_t out_stride_b, double* out, hipStream_t st) {
  const int64_t n = n_rz * m_series;
  if (n <= 0) return hipSuccess;
  k_finalize_multi<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(
      rzs, self_of, n_rz, m_series, static_cast<const Sums*>(partial), out_stride_b, out);
  return hipGetLastError();
}

size_t multi_sums_bytes() { return sizeof(Sums); }

hipError_t launch_finalize(const Realization* rzs, int64_t n_rz,
                           const Moments* partial, double* out, hipStream_t st) {
  if (n_rz <= 0) return hipSuccess;
  k_finalize<<<(unsigned)((n_rz + 255) / 256), 256, 0, st>>>(rzs, n_rz, partial, out);
  return hipGetLastError();
}

}  // namespace ccmk
