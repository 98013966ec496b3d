// Stages 2-3 of Alg. 1 on the GPU: the multiple-choice knapsack of Eq. 6 solved by
// Lagrangian bisection (Alg. 2), one search per item.
//
// For a multiplier lam the per-unit minimiser of w eps(b) + lam b is the highest
// vertex k of the lower convex hull of (b, eps(b)) with (double) w > lam * r_k,
// r_k the slope ratio of the hull edge into k (computed on the host).  Thresholds
// are fp64, the summed bits are integers, and the search returns the feasible
// iterate with the smallest multiplier (first one inside the tolerance band
// below the budget), so the result never exceeds the budget.
//
// Three things make a step cheap without changing a single verdict:
//   - (double) w > t is w > below(t), the largest fp32 number not above t, so units are compared in fp32, one
//     instruction per threshold, and counted in the lanes by the comparison's carry;
//   - a histogram over the leading bits of the fp32 pattern bounds the bit sum of any multiplier from both sides; while
//     the two bounds agree, no unit is read.  One wavefront evaluates the 63 multipliers the next six steps can visit at
//     once (a lane walks the midpoints to its node of the tree, so the multipliers are bit for bit those of Alg. 2);
//   - at the first step the bounds cannot decide, the units of the buckets that a threshold can still reach inside the
//     bracket [lo, hi] move to LDS and the remaining steps are evaluated exactly on those; what the other units add to
//     the bit sum follows from the histogram.
// Items of up to 32K units are searched by one workgroup that holds the units in registers and also writes the bit map
// and the counts the packing stage starts from (allocate_item_kernel: one launch instead of four to eight).  Longer
// items spread the passes over the units over many workgroups (slice_max_kernel, hist_kernel, gather_kernel, write_kernel); each
// of them takes the histogram's steps for itself, and the one that gathers an item's last open units the steps on those.
// Channel maps (128 units) take one wavefront (channel_allocate_kernel).
#include <algorithm>
#include <type_traits>

#include "rdkv_internal.h"
#include "wave_ops.h"

namespace rdkv {

namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;
constexpr int kMaxHull = 5;
constexpr int kThr = kMaxHull - 1;
constexpr int kBlockUnits = kPartBlock;   // units per block of the per-block tier counts
static_assert(kBlockUnits == kThreads, "a quarter of a round of allocate_item_kernel is one block");

struct SearchArgs {
  const float* w;
  const float* raw;            // the weights before the pooling, which the search's first launch then does; or null
  int32_t pool;                // keys of a pooling window (odd, at most 15)
  float pool_inv;              // 1 / pool
  uint8_t* bits;
  double r[kMaxHull];          // r[k-1]: threshold ratio into hull tier k
  int32_t tiers[kMaxHull];
  int32_t n_hull;
  int32_t max_iters;
  double need_frac;            // 1 - rel_tol
  double* lam_out;             // [items] or null: the multiplier of the returned allocation (NaN: no search ran)
  int32_t* iters_out;          // [items] or null: bisection steps taken
  int4* blk_counts;            // [blocks] out: units of the block in tiers 16, 8, 4, 2; or null
};
struct WholeItemArgs : SearchArgs {
  int32_t direct;              // allocate_item_kernel: steps taken on all units before the open ones are listed
  CountPost post;              // allocate_item_kernel, channel_allocate_kernel: where the host waits for the results, or nulls
};
// A kernel begins by reading some of its arguments out of cold memory, a line at a time: those that only some kernels have stand among
// the others for these alone.  (With them for all, eight items of 128K units in the many-workgroup form: slice_max_kernel 5.71 -> 5.86 us,
// hist_kernel 6.51 -> 6.81, gather_kernel 16.2 -> 16.5, write_kernel 4.9 -> 5.1.  Behind the batch, eight items of 4K to 16K units 14.2 ->
// 14.5, 16.4 -> 16.7, 22.9 -> 23.4.)
template <class Args>
struct Batched : Args {
  const int32_t* order;        // the items of this launch, or null: all of them as they stand
  Batch batch;
  __device__ __forceinline__ int item_of(int slot) const { return order ? __builtin_amdgcn_readfirstlane(order[slot]) : slot; }
};
using AllocArgs = Batched<WholeItemArgs>;

// largest fp32 number not above t (t >= 0): for fp32 w, (double) w > t exactly when w > below(t)
__device__ __forceinline__ float below(double t) {
  const float f = static_cast<float>(t);
  return static_cast<double>(f) > t ? __uint_as_float(__float_as_uint(f) - 1u) : f;
}

__device__ __forceinline__ int tier_slot(int b) { return b == 16 ? 0 : b == 8 ? 1 : b == 4 ? 2 : b == 2 ? 3 : -1; }

// c ? a : b of members of a structure (through the value: out of a plain selection the compiler makes one of two addresses, which puts
// the structure into memory)
__device__ __forceinline__ double either(bool c, double a, double b) {
  asm("" : "+v"(a), "+v"(b));
  return c ? a : b;
}

// ---- the search of one item ------------------------------------------------------------------------------------------
struct Problem {
  int32_t tiers[kMaxHull];
  int32_t step_bits[kThr];     // bits gained at threshold k (0 past the hull)
  double r[kThr];
  int nh, max_iters;
  long long base, B_int, need; // base: the bit sum with every unit in the lowest tier
  __device__ __forceinline__ Problem(const SearchArgs& a, int U, double budget) {
    nh = a.n_hull;
    max_iters = a.max_iters;
#pragma unroll
    for (int k = 0; k < kMaxHull; ++k) tiers[k] = a.tiers[k];
#pragma unroll
    for (int k = 0; k < kThr; ++k) {
      r[k] = a.r[k];
      step_bits[k] = k < nh - 1 ? a.tiers[k + 1] - a.tiers[k] : 0;
    }
    base = static_cast<long long>(tiers[0]) * U;
    B_int = static_cast<long long>(floor(budget * static_cast<double>(U)));
    need = static_cast<long long>(ceil(a.need_frac * static_cast<double>(B_int)));
  }
  // the tier every unit gets without a search, or -1
  // (the top tier by comparisons: an index known at run time puts the whole structure into memory)
  __device__ __forceinline__ int fill(int U) const {
    int top = tiers[0];
#pragma unroll
    for (int k = 1; k < kMaxHull; ++k) top = k < nh ? tiers[k] : top;
    if (B_int >= static_cast<long long>(top) * U) return top;
    if (nh == 1 || B_int < tiers[1]) return tiers[0];
    return -1;
  }
  // a unit is above threshold k of lam when it exceeds this
  __device__ __forceinline__ float thr(double lam, int k) const { return k < nh - 1 ? below(lam * r[k]) : INFINITY; }
  // the ratio of threshold lane % 4
  __device__ __forceinline__ double ratio_of_lane() const {
    static_assert(kThr == 4, "two bits of the lane");
    const bool odd = threadIdx.x & 1;
    return either(threadIdx.x & 2, either(odd, r[3], r[2]), either(odd, r[1], r[0]));
  }
  // bits of n units above threshold k
  __device__ __forceinline__ long long gain(int k, int n) const {
    return static_cast<long long>(static_cast<unsigned long long>(static_cast<unsigned>(step_bits[k])) * static_cast<unsigned>(n));
  }
  __device__ __forceinline__ int verdict(long long s) const { return s > B_int ? 0 : (s >= need ? 2 : 1); }
};

struct Search {
  double lo, hi, best;
  int have, it, done;
  // 0: over budget; 1: feasible, go on; 2: feasible and inside the band, stop
  __device__ __forceinline__ void take(int verdict, double lam) {
    ++it;
    if (verdict == 0) {
      lo = lam;
    } else {
      best = lam;
      have = 1;
      hi = lam;
      done = verdict == 2;
    }
  }
};

// LDS slot of histogram bucket b: one word of padding per 32, so that threads that own 8 or 32 consecutive buckets do not
// all hit the same banks
__host__ __device__ constexpr int hist_slot(int b) { return b + (b >> 5); }

// Histogram over the fp32 patterns of the positive units, ascending; suffix[b] = units in buckets >= b,
// suffix[BUCKETS] = 0.  bucket() is monotone in the unit.
// 256 buckets per factor of two below the largest unit's pattern (everything 2^-32 below it in bucket 0).
struct Anchored {
  static constexpr int kBuckets = 8192, kShift = 15, kWords = (hist_slot(kBuckets) + 4) / 4 * 4;
  uint32_t top;                // pattern of the largest unit
  __device__ __forceinline__ int bucket(uint32_t u) const {
    return u > top ? kBuckets : kBuckets - 1 - static_cast<int>(min((top - u) >> kShift, static_cast<uint32_t>(kBuckets - 1)));
  }
  // patterns of bucket b
  __device__ __forceinline__ uint32_t lowest(int b) const {
    const uint32_t d = ((static_cast<uint32_t>(kBuckets - b) << kShift) - 1u);      // largest top - u of the bucket
    return b == 0 || d >= top ? 0u : top - d;
  }
  __device__ __forceinline__ uint32_t highest(int b) const {
    const uint32_t d = static_cast<uint32_t>(kBuckets - 1 - b) << kShift;
    return d >= top ? 0u : top - d;
  }
};
// Steps of the search that the histogram decides, by one wavefront; returns with done set, max_iters reached or
// standing before a step it cannot decide.
__device__ __forceinline__ double readlane_f64(double v, int lane) {
  const uint64_t u = __double_as_longlong(v);
  const uint32_t lo = __builtin_amdgcn_readlane(static_cast<int>(u), lane), hi = __builtin_amdgcn_readlane(static_cast<int>(u >> 32), lane);
  return __longlong_as_double(static_cast<long long>((static_cast<uint64_t>(hi) << 32) | lo));
}
template <class Map>
__device__ __forceinline__ void steps_on_histogram(const Problem& P, const Map& map, const int* suffix, Search& S) {
  const int lane = threadIdx.x & 63, node = max(1, lane);
  const int depth = 31 - __clz(node);
  // bounds of the bit sum at lam: 0: over budget, 1: feasible, 2: feasible and inside the band, 3: cannot be decided here
  const auto judge = [&](double lam) __attribute__((always_inline)) {
    long long s_min = P.base, s_max = P.base;
#pragma unroll
    for (int k = 0; k < kThr; ++k) {
      // units in higher buckets than the threshold's are above it, units in lower ones are not
      const int b = map.bucket(__float_as_uint(P.thr(lam, k)));
      s_min += P.gain(k, suffix[hist_slot(min(b + 1, Map::kBuckets))]);
      s_max += P.gain(k, suffix[hist_slot(b)]);
    }
    if (s_min > P.B_int) return 0;
    if (s_max <= P.B_int && s_min >= P.need) return 2;
    return s_max < P.need ? 1 : 3;
  };
  if (S.lo == 0.0 && !S.done && S.it < P.max_iters) {
    // nothing was over budget so far: while that lasts the multipliers are hi / 2, hi / 4, ... (exact halves), a lane each
    const double lam = ldexp(S.hi, -(lane + 1));
    const int v = judge(lam);
    const unsigned long long other = __ballot(v != 1);
    const int run = min(other ? __ffsll(other) - 1 : 64, P.max_iters - S.it);    // feasible steps in a row
    if (run > 0) {
      S.it += run;
      S.have = 1;
      S.best = S.hi = readlane_f64(lam, run - 1);
    }
    if (run < 64 && S.it < P.max_iters) {
      const int next = __builtin_amdgcn_readlane(v, run);
      if (next == 3) return;
      S.take(next, readlane_f64(lam, run));
    }
  }
  while (!S.done && S.it < P.max_iters) {
    double lo = S.lo, hi = S.hi;                 // the bracket the search has at this lane's node
    for (int d = depth - 1; d >= 0; --d) {       // child 2 i: over budget (lo rises), child 2 i + 1: feasible (hi falls)
      const double mid = (lo + hi) * 0.5;
      if ((node >> d) & 1) hi = mid; else lo = mid;
    }
    const double lam = (lo + hi) * 0.5;
    const int v = judge(lam);
    const unsigned long long m_over = __ballot(v == 0), m_stop = __ballot(v == 2), m_open = __ballot(v == 3);
    int cur = 1, feasible = 0, it = S.it;        // feasible: the last node on the way with a feasible verdict
    bool open = false, done = false;
    while (cur < 64 && it < P.max_iters && !open && !done) {
      const unsigned long long bit = 1ull << cur;
      if (m_open & bit) {
        open = true;
      } else {
        ++it;
        if (m_over & bit) {
          cur = 2 * cur;
        } else {
          feasible = cur;
          done = (m_stop & bit) != 0;
          cur = 2 * cur + 1;
        }
      }
    }
    S.it = it;
    S.done = done;
    if (feasible) {
      S.best = readlane_f64(lam, feasible);
      S.have = 1;
    }
    if (cur < 64) {                              // the bracket at the node the walk stands before
      S.lo = readlane_f64(lo, cur);
      S.hi = readlane_f64(hi, cur);
    } else {                                     // the bracket after the walk's last node
      const int last = cur >> 1;
      const double at = readlane_f64(lam, last);
      S.lo = (cur & 1) ? readlane_f64(lo, last) : at;
      S.hi = (cur & 1) ? at : readlane_f64(hi, last);
    }
    if (open) return;
  }
}

// Where the search goes on after a step the histogram cannot decide, whichever way that step comes out: [lo, hi] contains
// its multiplier and every later one the histogram cannot decide either; a later multiplier above hi is feasible (and not
// inside the band), one below lo over budget.  A step can be undecided early, with a wide bracket, when its multiplier
// happens to lie next to the final one; the buckets open to the whole bracket then hold thousands of units (a gather of
// 13 us took 47), those open to [lo, hi] a few.
struct Hull { double lo, hi; };
__device__ __forceinline__ Hull bracket_of(const Search& S) { return Hull{S.lo, S.hi}; }
// (by one wavefront per outcome: `feasible` says which; gives lo or hi)
template <class Map>
__device__ __forceinline__ double narrow_hull(const Problem& P, const Map& map, const int* suffix, Search S, bool feasible) {
  S.take(feasible, (S.lo + S.hi) * 0.5);
  steps_on_histogram(P, map, suffix, S);
  return feasible ? S.lo : S.hi;
}
constexpr int kManyOpen = 4096;      // open units from which that pays
constexpr int kFewOpen = 1024;       // open units that a wavefront holds for the remaining steps

// In place: suffix[b] = sum of suffix[b ..]; suffix[BUCKETS] = 0.  All threads; barriers inside.
template <int BUCKETS>
__device__ __forceinline__ void suffix_sums(int* suffix, int* s_wave) {
  constexpr int kPer = BUCKETS / kThreads;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int v[kPer], local = 0;
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    v[i] = suffix[hist_slot(tid * kPer + i)];
    local += v[i];
  }
  const int below = static_cast<int>(wave_scan(static_cast<uint32_t>(local)));
  const int incl = __builtin_amdgcn_readlane(below, 63) - below + local;      // sum over this lane and the higher ones
  if (lane == 0) s_wave[wave] = incl;
  __syncthreads();
  int run = incl - local;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) run += w > wave ? s_wave[w] : 0;
#pragma unroll
  for (int i = kPer - 1; i >= 0; --i) {
    run += v[i];
    suffix[hist_slot(tid * kPer + i)] = run;
  }
  if (tid == 0) suffix[hist_slot(BUCKETS)] = 0;
  __syncthreads();
}

// The buckets that a threshold lam r_k can reach for lam in [h.lo, h.hi]: up to four disjoint ranges (rounded
// products and the bucket are monotone).  Units of other buckets keep their side of every threshold.
struct OpenBuckets {
  int a[kThr], b[kThr];            // range k: buckets a[k] .. b[k], empty when a[k] > b[k]
  __device__ __forceinline__ OpenBuckets() {}
  template <class Map>
  __device__ __forceinline__ OpenBuckets(const Problem& P, const Map& map, const Hull& h) {
    int prev = -1;
#pragma unroll
    for (int k = 0; k < kThr; ++k) {
      const bool used = k < P.nh - 1;
      b[k] = used ? min(map.bucket(__float_as_uint(P.thr(h.hi, k))), Map::kBuckets - 1) : prev;
      a[k] = used ? max(map.bucket(__float_as_uint(P.thr(h.lo, k))), prev + 1) : prev + 1;
      prev = max(prev, b[k]);
    }
  }
  // units in the open buckets
  __device__ __forceinline__ int count(const int* suffix) const {
    int n = 0;
#pragma unroll
    for (int k = 0; k < kThr; ++k) n += a[k] <= b[k] ? suffix[hist_slot(a[k])] - suffix[hist_slot(b[k] + 1)] : 0;
    return n;
  }
  // bit sum without the open buckets' units' gains
  __device__ __forceinline__ long long fixed(const Problem& P, const int* suffix) const {
    long long s = P.base;
#pragma unroll
    for (int k = 0; k < kThr; ++k) {
      if (k >= P.nh - 1) continue;
      int n = suffix[hist_slot(b[k] + 1)];
#pragma unroll
      for (int j = k + 1; j < kThr; ++j) n -= a[j] <= b[j] ? suffix[hist_slot(a[j])] - suffix[hist_slot(b[j] + 1)] : 0;
      s += P.gain(k, n);
    }
    return s;
  }
};
// the same ranges as fp32 patterns: unit u is in one when u - first <= span for some k
struct OpenPatterns {
  uint32_t first[kThr], span[kThr];
  template <class Map>
  __device__ __forceinline__ OpenPatterns(const OpenBuckets& o, const Map& map) {
#pragma unroll
    for (int k = 0; k < kThr; ++k) {
      const uint32_t lowest = max(map.lowest(o.a[k]), 1u), highest = map.highest(o.b[k]);   // (zero is above no threshold)
      const bool any = o.a[k] <= o.b[k] && lowest <= highest;
      first[k] = any ? lowest : 0xFFFFFFFFu;
      span[k] = any ? highest - lowest : 0u;
    }
  }
  __device__ __forceinline__ bool contains(float w) const {
    const uint32_t u = __float_as_uint(w);
    bool in = false;
#pragma unroll
    for (int k = 0; k < kThr; ++k) in |= u - first[k] <= span[k];
    return in;
  }
};

// Bits that a wavefront's units (N in each lane) gain above the thresholds, in every lane; n_units * 16 fits.  Counted in the lanes, two
// instructions per unit and threshold, and added up once: population counts of the comparison masks go through the scalar unit
// that the wavefronts of a SIMD share, and through scalar registers that 16 units and more do not have (one step on 8 units a
// thread 1.3 us, on 16 2.4).
// (as one block: a comparison's mask may be read two wait states after it, which the others' comparisons fill; out of additions of
// 32 units' comparisons the compiler made trees of selects that spilled.  t is uniform, and read two wait states earlier at the latest.)
__device__ __forceinline__ void count_above(float w, const float (&t)[4], int (&c)[4]) {
  uint64_t m1, m2, m3;
  asm volatile("v_cmp_lt_f32 vcc, %7, %11\n\t"
      "v_cmp_lt_f32_e64 %4, %8, %11\n\t"
      "v_cmp_lt_f32_e64 %5, %9, %11\n\t"
      "v_cmp_lt_f32_e64 %6, %10, %11\n\t"
      "v_addc_co_u32 %0, vcc, 0, %0, vcc\n\t"
      "v_addc_co_u32_e64 %1, %4, %1, 0, %4\n\t"
      "v_addc_co_u32_e64 %2, %5, %2, 0, %5\n\t"
      "v_addc_co_u32_e64 %3, %6, %3, 0, %6"
      : "+v"(c[0]), "+v"(c[1]), "+v"(c[2]), "+v"(c[3]), "=&s"(m1), "=&s"(m2), "=&s"(m3)
      : "s"(t[0]), "s"(t[1]), "s"(t[2]), "s"(t[3]), "v"(w)
      : "vcc");
}
// (used: how many of the N, in whole fours; uniform)
template <int N>
__device__ __forceinline__ int bits_above(const Problem& P, const float (&w)[N], const float (&t)[kThr], int used = N) {
  static_assert(kThr == 4, "the thresholds of count_above");
  // (a scalar that a lane was read into may be read two wait states later, which the compiler does not look after in a block)
  asm volatile("s_nop 1" :: "s"(t[0]), "s"(t[1]), "s"(t[2]), "s"(t[3]));
  __builtin_amdgcn_sched_barrier(0);
  int c[kThr] = {0, 0, 0, 0}, s = 0;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if (i > 0 && i % 4 == 0 && i >= used) break;
    count_above(w[i], t, c);
    __builtin_amdgcn_sched_barrier(0);     // (not all masks first: 32 units spilled)
  }
#pragma unroll
  for (int k = 0; k < kThr; ++k) s += __mul24(P.step_bits[k], c[k]);
  return __builtin_amdgcn_readlane(static_cast<int>(wave_scan(static_cast<uint32_t>(s))), 63);
}
// the thresholds of lam, a lane each (whole wavefronts)
__device__ __forceinline__ void thresholds(const Problem& P, double lam, float (&t)[kThr]) {
  const int own = __float_as_int(below(lam * P.ratio_of_lane()));
#pragma unroll
  for (int k = 0; k < kThr; ++k) t[k] = k < P.nh - 1 ? __int_as_float(__builtin_amdgcn_readlane(own, k)) : INFINITY;
}

// the sum of what the wavefronts have left in slots[kWaves], in every lane
__device__ __forceinline__ int sum_of_waves(const int* slots) {
  static_assert(kWaves == 16, "a row of lanes");
  return static_cast<int>(row_sum(static_cast<uint32_t>(slots[threadIdx.x & (kWaves - 1)])));
}

// The remaining steps, exactly, on n undecided units in LDS beside the decided ones' bit sum `fixed`.
// All threads; S is the same in all of them on entry and exit.  s_red: 2 kWaves ints.
__device__ __forceinline__ void steps_on_list(const Problem& P, const float* list, int n, long long fixed,
                                              const Hull& h, Search& S, int* s_red) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int parity = 0;
  while (!S.done && S.it < P.max_iters) {
    const double lam = (S.lo + S.hi) * 0.5;
    if (lam < h.lo || lam > h.hi) {      // uniform
      S.take(lam > h.hi, lam);
      continue;
    }
    float t[kThr];
#pragma unroll
    for (int k = 0; k < kThr; ++k) t[k] = P.thr(lam, k);
    int s = 0;                           // at most 32K units of 16 bits: fits
    for (int i0 = wave * 64; i0 < n; i0 += kThreads) {
      const int i = i0 + lane;
      const float w = i < n ? list[i] : 0.f;
#pragma unroll
      for (int k = 0; k < kThr; ++k) s += P.step_bits[k] * __popcll(__ballot(w > t[k]));
    }
    int* slots = s_red + parity * kWaves;        // alternating, so that one barrier per step is enough
    parity ^= 1;
    if (lane == 0) slots[wave] = s;
    __syncthreads();
    S.take(P.verdict(fixed + __builtin_amdgcn_readfirstlane(sum_of_waves(slots))), lam);
  }
}
// the same by one wavefront that holds up to 64 PER units in registers
template <int PER>
__device__ __forceinline__ void steps_in_wave(const Problem& P, const float (&w)[PER], long long fixed, const Hull& h, Search& S) {
  while (!S.done && S.it < P.max_iters) {
    const double lam = (S.lo + S.hi) * 0.5;
    if (lam < h.lo || lam > h.hi) {
      S.take(lam > h.hi, lam);
      continue;
    }
    long long s = fixed;
#pragma unroll
    for (int k = 0; k < kThr; ++k) {
      const float t = P.thr(lam, k);
      int c = 0;
#pragma unroll
      for (int i = 0; i < PER; ++i) c += __popcll(__ballot(w[i] > t));
      s += P.gain(k, c);
    }
    S.take(P.verdict(s), lam);
  }
}

// ... and the registers that n <= kFewOpen units take (a step compares all of them with every threshold)
template <class Unit>
__device__ __forceinline__ void steps_on_few(const Problem& P, int n, long long fixed, const Hull& h, Search& S, Unit&& unit) {
  const int lane = threadIdx.x & 63;
  const auto run = [&](auto& u, auto per) __attribute__((always_inline)) {
    constexpr int PER = decltype(per)::value;
#pragma unroll
    for (int i = 0; i < PER; ++i) u[i] = i * 64 + lane < n ? unit(i * 64 + lane) : 0.f;
    steps_in_wave<PER>(P, u, fixed, h, S);
  };
  if (n <= 64) {
    float u[1];
    run(u, std::integral_constant<int, 1>{});
  } else if (n <= 256) {
    float u[4];
    run(u, std::integral_constant<int, 4>{});
  } else {
    float u[16];
    run(u, std::integral_constant<int, 16>{});
  }
}

// The same by the whole workgroup, three steps at a time: wavefront i of the first eight evaluates the multiplier at node i of the tree of
// the next three steps' outcomes (steps_on_histogram has the numbering), then all of them walk down it.  One wavefront that took a
// step at a time needs 1.1 to 1.4 us each.  (Four wavefronts and two steps, sixteen and four: within 1 % of it.  The many-workgroup form,
// whose list is in memory and goes to one wavefront's registers without a barrier: 4 x 70K units 45.0 -> 46.0 us, 8 x 128K the same.)
// All threads; S is the same in all of them on entry and exit.  s_red: 2 kWaves ints.
constexpr int kNodes = 8;
template <int PER>
__device__ __forceinline__ void steps_in_tree(const Problem& P, const float* list, int n, long long fixed, const Hull& h, Search& S, int* s_red) {
  const int lane = threadIdx.x & 63;
  const int node = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  const int depth = 31 - __clz(max(1, node));
  static_assert(kNodes <= kWaves, "a wavefront per node");
  const bool works = node > 0 && node < kNodes;
  float w[PER];
  if (works) {
#pragma unroll
    for (int i = 0; i < PER; ++i) w[i] = i * 64 + lane < n ? list[i * 64 + lane] : 0.f;
  }
  int parity = 0;
  while (!S.done && S.it < P.max_iters) {
    int* slots = s_red + parity * kWaves;        // alternating, so that one barrier per round is enough
    parity ^= 1;
    if (works) {
      double lo = S.lo, hi = S.hi;
      for (int d = depth - 1; d >= 0; --d) {
        const double mid = (lo + hi) * 0.5;
        if ((node >> d) & 1) hi = mid; else lo = mid;
      }
      const double lam = (lo + hi) * 0.5;
      int v = lam > h.hi ? 1 : 0;          // outside the hull (uniform)
      if (lam >= h.lo && lam <= h.hi) {
        float t[kThr];
        thresholds(P, lam, t);
        v = P.verdict(fixed + bits_above(P, w, t));
      }
      if (lane == 0) slots[node] = v;
    }
    __syncthreads();
    for (int cur = 1; cur < kNodes && !S.done && S.it < P.max_iters;) {
      const int verdict = slots[cur];
      S.take(verdict, (S.lo + S.hi) * 0.5);
      cur = 2 * cur + (verdict != 0);
    }
  }
}
__device__ __forceinline__ void steps_on_short_list(const Problem& P, const float* list, int n, long long fixed, const Hull& h, Search& S, int* s_red) {
  if (n <= 64) steps_in_tree<1>(P, list, n, fixed, h, S, s_red);
  else if (n <= 256) steps_in_tree<4>(P, list, n, fixed, h, S, s_red);
  else if (n <= 512) steps_in_tree<8>(P, list, n, fixed, h, S, s_red);
  else steps_in_tree<16>(P, list, n, fixed, h, S, s_red);
}

__device__ __forceinline__ void report(const SearchArgs& a, int item, bool searched, const Search& S) {
  if (a.lam_out) a.lam_out[item] = searched && S.have ? S.best : __longlong_as_double(0x7FF8000000000000ll);
  if (a.iters_out) a.iters_out[item] = searched ? S.it : 0;
}

// A round of 64 units: the tier of this lane's unit, and (in every lane) how many of the wavefront's units are above each
// threshold.
__device__ __forceinline__ int tier_of(const Problem& P, float w, const float (&t)[kThr], int (&above)[kThr]) {
  int b = P.tiers[0];
#pragma unroll
  for (int k = 0; k < kThr; ++k) {                                       // thresholds ascend
    const bool up = w > t[k];
    b = up ? P.tiers[k + 1] : b;
    above[k] = __popcll(__ballot(up));
  }
  return b;
}
// counts above the thresholds of a block with n units -> counts per stored tier
__device__ __forceinline__ int4 tier_counts(const Problem& P, int n, const int4& above) {
  const int c[kMaxHull + 1] = {n, above.x, above.y, above.z, above.w, 0};
  int out[4] = {0, 0, 0, 0};
#pragma unroll
  for (int i = 0; i < kMaxHull; ++i) {
    const int in = i < P.nh ? c[i] - (i < P.nh - 1 ? c[i + 1] : 0) : 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) out[k] += P.tiers[i] == (16 >> k) ? in : 0;
  }
  return make_int4(out[0], out[1], out[2], out[3]);
}

// four consecutive units at any 4-byte boundary, and their four bytes of the bit map at any address
struct __attribute__((packed, aligned(4))) Units4 { float v[4]; };
struct __attribute__((packed, aligned(1))) Bytes4 { uint32_t v; };

// AvgPool1d(pool, stride 1, zero padding pool / 2, divisor pool) of raw weights in LDS (pool_kernel in the weights' file is the
// launch of its own), added in the same order and divided to the same bits: the correctly rounded quotient from the correctly
// rounded reciprocal and one exact remainder (Markstein, IBM J. Res. Dev. 34, 1990), by division where the remainder could
// underflow or is none.
constexpr int kMostRadius = 7;
__device__ __forceinline__ void pool_quotients(const SearchArgs& a, float (&s)[4]) {
  const float n = static_cast<float>(a.pool);
  // (sums of weights: not negative, so that their patterns are ordered as they are; less one, a zero, which is its own
  // quotient, comes to the other end: with 97 in 100 weights zero eight items of 32K units 18.8 -> 17.7 us)
  const uint32_t u[4] = {__float_as_uint(s[0]), __float_as_uint(s[1]), __float_as_uint(s[2]), __float_as_uint(s[3])};
  const uint32_t least = min(min(min(u[0] - 1u, u[1] - 1u), u[2] - 1u), u[3] - 1u), most = max(max(max(u[0], u[1]), u[2]), u[3]);
  float q[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float q0 = s[e] * a.pool_inv;
    q[e] = __builtin_fmaf(__builtin_fmaf(-q0, n, s[e]), a.pool_inv, q0);
  }
  if (__builtin_expect(__any(least < __float_as_uint(1e-25f) - 1u || most > __float_as_uint(1e30f)), 0)) {
#pragma unroll
    for (int e = 0; e < 4; ++e) q[e] = s[e] / n;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) s[e] = q[e];
}
// four units of a window of five from the eight weights under it
__device__ __forceinline__ void pool_five(const SearchArgs& a, const float (&t)[8], float (&v)[4]) {
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = (((t[e] + t[e + 1]) + t[e + 2]) + t[e + 3]) + t[e + 4];
  pool_quotients(a, v);
}
// ... of any window, the first of which starts at w[0]
__device__ __forceinline__ void pool_any(const SearchArgs& a, const float* w, float (&v)[4]) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    v[e] = 0.f;
    for (int k = 0; k < a.pool; ++k) v[e] += w[e + k];
  }
  pool_quotients(a, v);
}

// ---- one workgroup per item: up to 1024 REG units in registers ------------------------------------------------------
// Thread t holds units 4096 j + 4 t .. + 3, so four wavefronts make one block of the per-block counts.  What bounds it:
// one compute unit works on an item, through the latency of its loads and about fifteen barriers and then the number of
// instructions per unit and pass (load, histogram, gather, write).  Measured against fp64 comparisons and one step at a time: 4K
// units 31 -> 8.4 us, 32K units (94 us in five kernels) -> 24 us, both with the counting kernels (10 us) gone; with the pooling,
// which had a launch of its own, 9.5 and 28.  By time stamps, 8K units were 1.7 us of pooling, 3.9 of histogram and its steps, 7.6 of
// the other steps and 1.5 of the map, 32K units 5.1, 7.2, 7.5 and 4.0: with a class of 8K units whose steps are all taken in
// registers, population counts turned into carries, and one range check per four quotients, eight items of 8K units 20.7 -> 14.0 us,
// of 4K 9.5 -> 8.9, of 16K 2.3 less, of 32K 1.5 less; 128 items of 20K 31.1 -> 28.7.
constexpr int kItemListCap = 24576;        // units of open buckets in LDS (96 KB beside 34 KB of histogram)
template <int REG>
constexpr size_t kItemLds = Anchored::kWords * sizeof(int) + (REG <= 8 ? REG / 4 * kWaves * 2 * sizeof(uint32_t) : kItemListCap * sizeof(float));

// Result `i` of an item for the host, which watches the words (the lanes that have one come here).
__device__ __forceinline__ void post_word(uint64_t* words, int64_t i, uint32_t tag, uint32_t value) {
  __hip_atomic_store(words + i, (static_cast<uint64_t>(tag) << 32) | value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

template <int REG>
__global__ __launch_bounds__(kThreads) void allocate_item_kernel(AllocArgs a) {
  constexpr int kQ = REG / 4;
  extern __shared__ __align__(16) unsigned char smem[];
  int* s_hist = reinterpret_cast<int*>(smem);
  float* s_list = reinterpret_cast<float*>(s_hist + Anchored::kWords);      // [kItemListCap]
  uint32_t* s_cnt = reinterpret_cast<uint32_t*>(s_list);                        // [kQ][kWaves][2], after the search
  __shared__ int s_wave[kWaves], s_red[2 * kWaves], s_n;
  __shared__ float s_max[kWaves];
  __shared__ Search s_search;
  __shared__ Hull s_hull;
  const int item = a.item_of(blockIdx.x);
  const ItemOf it(a.batch, item);
  const int U = it.T;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float* w = a.w + it.off;
  uint8_t* __restrict__ bits = a.bits + it.off;
  const int used = 4 * ((U + 4 * kThreads - 1) / (4 * kThreads));     // of a thread's units
  float v[REG];                            // units past the end read as 0: never above a threshold
  if (a.raw) w = a.raw + it.off;
#pragma unroll
  for (int j = 0; j < kQ; ++j) {
    const int u0 = 4 * (j * kThreads + tid);
    if (u0 + 3 < U) {
      const Units4 x = *reinterpret_cast<const Units4*>(w + u0);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[4 * j + e] = x.v[e];
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[4 * j + e] = u0 + e < U ? w[u0 + e] : 0.f;
    }
  }
  if (a.raw) {
    // through LDS, which nothing else uses yet, for the neighbours' sake: unit u at s_raw[kPad + u], zeros around them
    constexpr int kPad = 8;
    static_assert(kPad > kMostRadius && kItemLds<REG> >= (REG * kThreads + 2 * kPad) * sizeof(float), "an item and its window's ends");
    float* s_raw = reinterpret_cast<float*>(smem);
    if (tid < kPad) s_raw[tid] = s_raw[kPad + (U + 3) / 4 * 4 + tid] = 0.f;
#pragma unroll
    for (int j = 0; j < kQ; ++j) {
      const int u0 = 4 * (j * kThreads + tid);
      if (u0 < U) *reinterpret_cast<float4*>(s_raw + kPad + u0) = make_float4(v[4 * j], v[4 * j + 1], v[4 * j + 2], v[4 * j + 3]);
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kQ; ++j) {
      const int u0 = 4 * (j * kThreads + tid);
      if (u0 < U) {
        float x[4];
        if (a.pool == 5) {                 // (uniform)
          const float2 lo = *reinterpret_cast<const float2*>(s_raw + kPad + u0 - 2), hi = *reinterpret_cast<const float2*>(s_raw + kPad + u0 + 4);
          const float t[8] = {lo.x, lo.y, v[4 * j], v[4 * j + 1], v[4 * j + 2], v[4 * j + 3], hi.x, hi.y};
          pool_five(a, t, x);
        } else {
          pool_any(a, s_raw + kPad + u0 - a.pool / 2, x);
        }
        const bool inside = 4 * (j + 1) * kThreads <= U;      // (uniform)
#pragma unroll
        for (int e = 0; e < 4; ++e) v[4 * j + e] = inside || u0 + e < U ? x[e] : 0.f;
      }
    }
    __syncthreads();
  }
  for (int i = tid; i < Anchored::kWords / 4; i += kThreads) reinterpret_cast<int4*>(s_hist)[i] = make_int4(0, 0, 0, 0);
  const Problem P(a, U, it.budget);
  const int fill = U > 0 ? P.fill(U) : P.tiers[0];
  Search S{0.0, 0.0, 0.0, 0, 0, 0};
  float t[kThr];
#pragma unroll
  for (int k = 0; k < kThr; ++k) t[k] = INFINITY;

  if (fill < 0) {
    float mx = 0.f;
#pragma unroll
    for (int j = 0; j < REG; ++j) mx = fmaxf(mx, v[j]);
    mx = wave_max(mx);
    if (lane == 0) s_max[wave] = mx;
    __syncthreads();
    mx = s_max[0];
#pragma unroll
    for (int i = 1; i < kWaves; ++i) mx = fmaxf(mx, s_max[i]);
    const Anchored map{__float_as_uint(mx)};
#pragma unroll
    for (int j = 0; j < REG; ++j)
      if (v[j] > 0.f) atomicAdd(&s_hist[hist_slot(map.bucket(__float_as_uint(v[j])))], 1);
    __syncthreads();
    suffix_sums<Anchored::kBuckets>(s_hist, s_wave);
    S.hi = static_cast<double>(mx);

    while (true) {
      if (wave == 0) {
        steps_on_histogram(P, map, s_hist, S);
        if (lane == 0) {
          s_search = S;
          s_n = 0;
        }
      }
      __syncthreads();
      S = s_search;
      if (S.done || S.it >= P.max_iters) break;
      // the histogram cannot decide the next step
      // Up to 8K units the other steps are taken on all of them, 1 us each; up to 16K the first a.direct of them, 1.4 us each (see
      // launch_short_items).  An item has 0 to 5 of them left.  The open buckets, the list and its few units' steps take 6 to 7 us: 5000
      // units 19.2 -> 13.4 us in all, 8K 21.6 -> 15.7 (of eight items; a launch of them takes 2 us, events around it 2 more).  With 32
      // units per thread a step costs 2.2 us, and the slowest of 128 items takes five: 34.2 -> 35.5.
      if constexpr (REG <= 16) {
        int parity = 0;
        for (int taken = 0; (REG <= 8 || taken < a.direct) && !S.done && S.it < P.max_iters; ++taken) {
          const double lam = (S.lo + S.hi) * 0.5;
          thresholds(P, lam, t);
          const int c = bits_above(P, v, t, used);
          int* slots = s_red + parity * kWaves;        // alternating, so that one barrier per step is enough
          parity ^= 1;
          if (lane == 0) slots[wave] = c;
          __syncthreads();
          S.take(P.verdict(P.base + __builtin_amdgcn_readfirstlane(sum_of_waves(slots))), lam);
        }
        if (REG <= 8 || S.done || S.it >= P.max_iters) break;
        __syncthreads();                   // s_red is not read any more
      }
      Hull hull = bracket_of(S);
      OpenBuckets open(P, map, hull);
      int n = open.count(s_hist);
      if (n > kManyOpen) {
        if (wave < 2) {
          const double end = narrow_hull(P, map, s_hist, S, wave == 0);
          if (lane == 0) (wave == 0 ? s_hull.lo : s_hull.hi) = end;
        }
        __syncthreads();
        hull = s_hull;
        open = OpenBuckets(P, map, hull);
        n = open.count(s_hist);
      }
      if (n <= kItemListCap) {
        const OpenPatterns pat(open, map);
        uint32_t mine = 0;                 // which of this thread's units
#pragma unroll
        for (int j = 0; j < REG; ++j) mine |= pat.contains(v[j]) ? 1u << j : 0u;
        const int own = __popc(mine), incl = static_cast<int>(wave_scan(static_cast<uint32_t>(own)));
        int base = 0;
        if (lane == 63) base = atomicAdd(&s_n, incl);
        float* dst = s_list + __builtin_amdgcn_readlane(base, 63) + incl - own;
#pragma unroll
        for (int j = 0; j < REG; ++j)
          if ((mine >> j) & 1) *dst++ = v[j];
        __syncthreads();
        const long long fixed = open.fixed(P, s_hist);
        if (n <= kFewOpen) steps_on_short_list(P, s_list, n, fixed, hull, S, s_red);
        else steps_on_list(P, s_list, n, fixed, hull, S, s_red);
        break;
      }
      // too many for LDS: this one step on all units, then the histogram again with half the bracket
      const double lam = (S.lo + S.hi) * 0.5;
      thresholds(P, lam, t);
      const int c = bits_above(P, v, t, used);
      if (lane == 0) s_red[wave] = c;
      __syncthreads();
      long long s = P.base;
      for (int i = 0; i < kWaves; ++i) s += s_red[i];
      S.take(P.verdict(s), lam);
      __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < kThr; ++k) t[k] = S.have ? P.thr(S.best, k) : INFINITY;
  }
  if (tid == 0) report(a, item, fill < 0, S);

  // ---- the bit map, and the tier counts of every block -----------------------------------------------------------
  const int nblk = (U + kBlockUnits - 1) / kBlockUnits;
  if (fill >= 0) {
    for (int u = tid; u < U; u += kThreads) bits[u] = static_cast<uint8_t>(fill);
    if (a.blk_counts && tid < nblk) {
      const int n = min(kBlockUnits, U - tid * kBlockUnits);
      a.blk_counts[it.blk0 + tid] =
          make_int4(fill == 16 ? n : 0, fill == 8 ? n : 0, fill == 4 ? n : 0, fill == 2 ? n : 0);
    }
    if (a.post.counts && tid < 4) post_word(a.post.counts, 4 * static_cast<int64_t>(item) + tid, a.post.tag, fill == (16 >> tid) ? U : 0);
    return;
  }
  __syncthreads();                         // the list is not read any more
  // (Tiers are one bit each: a byte per unit counts them, eight bits per tier up to 32 lanes.  Only where somebody wants the counts: a
  // search by itself, eight items of 4K units 9.65 -> 9.3 us, of 20K 20.1 -> 19.7, of 32K 21.8 -> 21.1.)
#pragma unroll
  for (int j = 0; j < kQ; ++j) {
    const int u0 = 4 * (j * kThreads + tid);
    if (4 * j * kThreads < U) {            // (uniform)
      uint32_t packed = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        uint32_t b = static_cast<uint32_t>(P.tiers[0]);
#pragma unroll
        for (int k = 0; k < kThr; ++k) b = v[4 * j + e] > t[k] ? static_cast<uint32_t>(P.tiers[k + 1]) : b;      // thresholds ascend
        packed |= b << (8 * e);
      }
      if (u0 + 3 < U) {
        reinterpret_cast<Bytes4*>(bits + u0)->v = packed;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (u0 + e < U) bits[u0 + e] = static_cast<uint8_t>(packed >> (8 * e));
          else packed &= ~(0xFFu << (8 * e));
        }
      }
      if (a.blk_counts) {
        uint32_t n = 0;                    // in tiers 16, 8, 4, 2
#pragma unroll
        for (int k = 0; k < 4; ++k) n |= static_cast<uint32_t>(__popc(packed & (0x10101010u >> k))) << (8 * k);
        n = row_pair_sum(n);
        if ((lane & 31) == 31) s_cnt[(j * kWaves + wave) * 2 + (lane >> 5)] = n;
      }
    }
  }
  if (a.blk_counts) {
    __syncthreads();
    if (wave > 0) return;
    static_assert(REG <= 32, "a lane per block, and counts of 16 bits");
    uint32_t even = 0, odd = 0;            // tiers 16 and 4; 8 and 2
    if (tid < nblk) {                      // block tid: wavefronts 4 tid .. 4 tid + 3 of the rounds in one line
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const uint32_t x = s_cnt[8 * tid + i];
        even += x & 0x00FF00FFu;
        odd += (x >> 8) & 0x00FF00FFu;
      }
      a.blk_counts[it.blk0 + tid] = make_int4(even & 0xFFFF, odd & 0xFFFF, even >> 16, odd >> 16);
    }
    if (a.post.counts) {
      even = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(wave_scan(even)), 63));
      odd = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(wave_scan(odd)), 63));
      const uint32_t pair = tid & 1 ? odd : even;
      if (tid < 4) post_word(a.post.counts, 4 * static_cast<int64_t>(item) + tid, a.post.tag, tid & 2 ? pair >> 16 : pair & 0xFFFF);
    }
  }
}
constexpr int kItemUnits = 32 * kThreads;   // longest item of that kernel

// ---- longer items: the passes over the units on many workgroups -------------------------------------------------
// Beyond 32K units the registers of one compute unit no longer hold an item.  Measured, 8 items of 128K units: 98 to 255
// us in six kernels -> 32 us in four, pooling included; what is left is the latency of a hand-over to the last workgroup and of the
// dependent steps.
// An item's weights read as aligned 16-byte quads.  Quad q covers units 4 q - a .. 4 q - a + 3,
// a = how many floats the item's first weight sits past a 16-byte boundary; units outside [0, U) read as 0 (never above
// a threshold).  The first and the last quad are read element by element (their neighbours may lie outside the array).
struct Quads {
  const float* w;
  int a, U, nq;
  __device__ Quads(const float* w_, int U_) : w(w_), U(U_) {
    a = static_cast<int>((reinterpret_cast<uintptr_t>(w_) >> 2) & 3);
    nq = (U_ + a + 3) >> 2;
  }
  __device__ __forceinline__ void load(int q, float (&v)[4]) const {
    const int u0 = 4 * q - a;
    if (q > 0 && q + 1 < nq) {
      const float4 t = *reinterpret_cast<const float4*>(w + u0);
      v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = (q < nq && u0 + j >= 0 && u0 + j < U) ? w[u0 + j] : 0.0f;
    }
  }
  // this workgroup's quads
  __device__ __forceinline__ void slice(int slices, int* q0, int* q1) const {
    const int per = (nq + slices - 1) / slices;
    *q0 = min(nq, static_cast<int>(blockIdx.x) * per);
    *q1 = min(nq, *q0 + per);
  }
};

constexpr int kMostSlices = 16;              // workgroups that share an item
constexpr int kMostMaxima = 2 * kMostSlices; // workgroups that share its first pass
static_assert(kMostMaxima <= 64, "a lane each");
constexpr int kListCap = 24576;             // undecided units of an item (96 KB of LDS in the exact steps)
struct SearchState {
  Search s;                                 // the search's end
  int32_t n_list, arrive, fill;             // fill: >= 0: the tier of every unit
};
struct MultiArgs {
  Batched<SearchArgs> a;
  // per item of the launch (grid row), not of the batch
  int32_t* hist;        // [rows][kBuckets], zero on entry
  SearchState* state;   // [rows], zero on entry
  float* list;          // [rows][kListCap]
  float* slice_max;     // [rows][maxima]
  int32_t slices, maxima;
};

// Called by all threads of a workgroup after their stores and atomics of a pass: true in the workgroup that is the last
// of `count` to call it.  What the others wrote with agent-scope accesses can then be read with agent-scope loads.
__device__ __forceinline__ bool last_to_arrive(int32_t* counter, int count, int* s_flag) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0)
    *s_flag = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == count - 1;
  __syncthreads();
  return *s_flag != 0;
}
template <class T>
__device__ __forceinline__ T load_agent(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The largest unit of every slice, which anchors the histograms (over the full range of fp32 they had 32768 buckets at a
// quarter of the resolution: hist_kernel 21 us, gather_kernel 20 at 8 x 128K units), and zeros for the next kernels.
// POOL: raw weights are pooled on the way and written for the next kernels (8 x 128K units: 5.8 us, as two launches 5.1 + 4.7).
template <bool POOL>
__global__ __launch_bounds__(kThreads) void slice_max_kernel(MultiArgs m, float* pooled, uint4* clear, int64_t n_clear) {
  constexpr int kRound = 4 * kThreads;
  __shared__ __align__(16) float s_raw[POOL ? kRound + 2 * kMostRadius + 2 : 4];
  __shared__ float s_max[kWaves];
  const int row = blockIdx.y, tid = threadIdx.x;
  const ItemOf it(m.a.batch, m.a.item_of(row));
  const int64_t step = static_cast<int64_t>(gridDim.x) * gridDim.y * kThreads;
  for (int64_t i = (static_cast<int64_t>(row) * gridDim.x + blockIdx.x) * kThreads + tid; i < n_clear; i += step)
    clear[i] = make_uint4(0, 0, 0, 0);
  // whole rounds per workgroup, so that a slice starts at a multiple of four
  const int rounds = (it.T + kRound - 1) / kRound, per = (rounds + static_cast<int>(gridDim.x) - 1) / static_cast<int>(gridDim.x);
  const int u_first = min(it.T, static_cast<int>(blockIdx.x) * per * kRound), u_last = min(it.T, u_first + per * kRound);
  float mx = 0.f;
  if constexpr (POOL) {
    const float* raw = m.a.raw + it.off;
    float* out = pooled + it.off;
    const int radius = m.a.pool / 2;
    for (int u0 = u_first; u0 < u_last; u0 += kRound) {
      float v[5];
#pragma unroll
      for (int j = 0; j < 5; ++j) {
        const int u = u0 - radius + j * kThreads + tid;
        v[j] = (j < 4 || tid < 2 * radius) && u >= 0 && u < it.T ? raw[u] : 0.f;
      }
      __syncthreads();                     // the round before is used up
#pragma unroll
      for (int j = 0; j < 5; ++j)
        if (j < 4 || tid < 2 * radius) s_raw[j * kThreads + tid] = v[j];
      __syncthreads();
      float x[4];
      if (m.a.pool == 5) {                 // (uniform)
        const float4 lo = *reinterpret_cast<const float4*>(s_raw + 4 * tid), hi = *reinterpret_cast<const float4*>(s_raw + 4 * tid + 4);
        const float t[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
        pool_five(m.a, t, x);
      } else {
        pool_any(m.a, s_raw + 4 * tid, x);
      }
      const int u = u0 + 4 * tid;
      if (u + 3 < u_last) {
        *reinterpret_cast<Units4*>(out + u) = Units4{{x[0], x[1], x[2], x[3]}};
        mx = fmaxf(mx, fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])));
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (u + e < u_last) {
            out[u + e] = x[e];
            mx = fmaxf(mx, x[e]);
          }
      }
    }
  } else {
    const float* w = m.a.w + it.off;
    for (int u = u_first + 4 * tid; u < u_last; u += kRound) {
      if (u + 3 < u_last) {
        const Units4 x = *reinterpret_cast<const Units4*>(w + u);
        mx = fmaxf(mx, fmaxf(fmaxf(x.v[0], x.v[1]), fmaxf(x.v[2], x.v[3])));
      } else {
        for (int e = 0; u + e < u_last; ++e) mx = fmaxf(mx, w[u + e]);
      }
    }
  }
  mx = wave_max(mx);
  if ((tid & 63) == 0) s_max[tid >> 6] = mx;
  __syncthreads();
  if (tid < 64) {
    mx = wave_max(tid < kWaves ? s_max[tid] : 0.f);
    if (tid == 0) m.slice_max[row * m.maxima + blockIdx.x] = mx;
  }
}

// every slice adds its units to the item's histogram
constexpr size_t kHistLds = Anchored::kWords * sizeof(int);
__device__ __forceinline__ float largest_unit(const MultiArgs& m, int row) {      // (before wave_max)
  const int lane = threadIdx.x & 63;
  return lane < m.maxima ? m.slice_max[row * m.maxima + lane] : 0.f;
}
__global__ __launch_bounds__(kThreads) void hist_kernel(MultiArgs m) {
  extern __shared__ __align__(16) unsigned char smem[];
  int* s_hist = reinterpret_cast<int*>(smem);
  const Batched<SearchArgs>& a = m.a;
  const int row = blockIdx.y;
  const ItemOf it(a.batch, a.item_of(row));
  const int U = it.T;
  const int tid = threadIdx.x;
  const Quads quads(a.w + it.off, U);
  int q0, q1;
  quads.slice(m.slices, &q0, &q1);
  float mx = largest_unit(m, row);
  float wv[4] = {0.f, 0.f, 0.f, 0.f};
  if (q0 + tid < q1) quads.load(q0 + tid, wv);
  const Problem P(a, U, it.budget);
  if (U <= 0 || P.fill(U) >= 0) return;
  for (int i = tid; i < Anchored::kWords / 4; i += kThreads) reinterpret_cast<int4*>(s_hist)[i] = make_int4(0, 0, 0, 0);
  mx = wave_max(mx);
  const Anchored map{__float_as_uint(mx)};
  __syncthreads();
  for (int q = q0 + tid; q < q1;) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (wv[e] > 0.f) atomicAdd(&s_hist[hist_slot(map.bucket(__float_as_uint(wv[e])))], 1);
    q += kThreads;
    if (q < q1) quads.load(q, wv);
  }
  __syncthreads();
  int32_t* gh = m.hist + static_cast<int64_t>(row) * Anchored::kBuckets;
  for (int i = tid; i < Anchored::kBuckets; i += kThreads)
    if (s_hist[hist_slot(i)] != 0) atomicAdd(gh + i, s_hist[hist_slot(i)]);
}

// Every slice takes the steps the histogram decides for itself (the last workgroup of the kernel before did, for all: it waited for
// the others' sums and its state went through memory: hist 13.3 + gather 10.5 us at 8 x 128K units, now 6.5 + 15.6), then appends
// its units of open buckets to the item's list; the last one takes the other steps.
constexpr size_t kGatherLds = Anchored::kWords * sizeof(int) + kListCap * sizeof(float);
__global__ __launch_bounds__(kThreads) void gather_kernel(MultiArgs m) {
  extern __shared__ __align__(16) unsigned char smem[];
  int* s_hist = reinterpret_cast<int*>(smem);
  float* s_list = reinterpret_cast<float*>(s_hist + Anchored::kWords);      // [kListCap]
  __shared__ int s_wave[kWaves], s_n, s_base, s_above[kThr], s_flag, s_red[2 * kWaves];
  __shared__ Search s_search;
  __shared__ Hull s_hull;
  const Batched<SearchArgs>& a = m.a;
  const int row = blockIdx.y, item = a.item_of(row);
  const ItemOf it(a.batch, item);
  const int U = it.T;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  SearchState& st = m.state[row];
  const Quads quads(a.w + it.off, U);
  int q0, q1;
  quads.slice(m.slices, &q0, &q1);
  constexpr int kPer = Anchored::kBuckets / kThreads;
  int h[kPer];
  const int32_t* gh = m.hist + static_cast<int64_t>(row) * Anchored::kBuckets;
  float mx = largest_unit(m, row);
#pragma unroll
  for (int k = 0; k < kPer; ++k) h[k] = gh[tid + k * kThreads];
  float w0[4] = {0.f, 0.f, 0.f, 0.f};      // the slice's first round, on its way during the steps
  if (q0 + tid < q1) quads.load(q0 + tid, w0);
  const Problem P(a, U, it.budget);
  const int fill = U > 0 ? P.fill(U) : P.tiers[0];
  if (fill >= 0) {
    if (blockIdx.x == 0 && tid == 0) {
      st.fill = fill;
      st.s = Search{0.0, 0.0, 0.0, 0, 0, 1};
      report(a, item, false, st.s);
    }
    return;
  }
#pragma unroll
  for (int k = 0; k < kPer; ++k) s_hist[hist_slot(tid + k * kThreads)] = h[k];
  mx = wave_max(mx);
  const Anchored map{__float_as_uint(mx)};
  if (tid == 0) s_n = 0;
  __syncthreads();
  suffix_sums<Anchored::kBuckets>(s_hist, s_wave);
  if (wave < 2) {                        // two wavefronts, the same steps
    Search T{0.0, static_cast<double>(mx), 0.0, 0, 0, 0};
    steps_on_histogram(P, map, s_hist, T);
    T.done = T.done || T.it >= P.max_iters;
    const Hull bracket = bracket_of(T);
    const bool many = !T.done && OpenBuckets(P, map, bracket).count(s_hist) > kManyOpen;
    const double end = many ? narrow_hull(P, map, s_hist, T, wave == 0) : wave == 0 ? bracket.lo : bracket.hi;
    if (lane == 0) (wave == 0 ? s_hull.lo : s_hull.hi) = end;
    if (tid == 0) s_search = T;
  }
  __syncthreads();
  Search S = s_search;
  if (S.done) {
    if (blockIdx.x == 0 && tid == 0) {
      st.fill = -1;
      st.s = S;
      report(a, item, true, S);
    }
    return;
  }
  const Hull hull = s_hull;
  const OpenBuckets open(P, map, hull);
  const int n = open.count(s_hist);
  if (n > kListCap && blockIdx.x != 0) return;
  if (n <= kListCap) {
    float* gl = m.list + static_cast<int64_t>(row) * kListCap;
    const OpenPatterns pat(open, map);
    for (int qw = q0 + wave * 64; qw < q1; qw += kThreads) {
      float wv[4] = {w0[0], w0[1], w0[2], w0[3]};
      if (qw != q0 + wave * 64) {
#pragma unroll
        for (int e = 0; e < 4; ++e) wv[e] = 0.f;
        if (qw + lane < q1) quads.load(qw + lane, wv);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool in = pat.contains(wv[e]);
        const unsigned long long mask = __ballot(in);
        if (mask) {
          int base = 0;
          if (lane == 0) base = atomicAdd(&s_n, __popcll(mask));
          base = __builtin_amdgcn_readfirstlane(base) + __popcll(mask & ((1ull << lane) - 1ull));
          if (in) s_list[base] = wv[e];
        }
      }
    }
    __syncthreads();
    const int mine = s_n;
    if (tid == 0) s_base = mine ? atomicAdd(&st.n_list, mine) : 0;
    __syncthreads();
    for (int i = tid; i < mine; i += kThreads)
      __hip_atomic_store(gl + s_base + i, s_list[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (!last_to_arrive(&st.arrive, m.slices, &s_flag)) return;
    const long long fixed = open.fixed(P, s_hist);
    if (n <= kFewOpen) {
      if (wave == 0) {
        steps_on_few(P, n, fixed, hull, S, [&](int i) { return load_agent(gl + i); });
        if (lane == 0) s_search = S;
      }
      __syncthreads();
      S = s_search;
    } else {
      for (int i = tid; i < n; i += kThreads) s_list[i] = load_agent(gl + i);
      __syncthreads();
      steps_on_list(P, s_list, n, fixed, hull, S, s_red);
    }
  } else {
    // More than the list holds (weights all alike, or in a band of a few ulp): every step on all units, one workgroup.
    // 8 items of 128K units, one value, 64 steps: 820 us (with fp64 comparisons 1470); a band of 1e-3, 20 steps: 190 (440).
    while (!S.done && S.it < P.max_iters) {
      const double lam = (S.lo + S.hi) * 0.5;
      float t[kThr];
#pragma unroll
      for (int k = 0; k < kThr; ++k) t[k] = P.thr(lam, k);
      int c[kThr] = {0, 0, 0, 0};
      for (int qw = wave * 64; qw < quads.nq; qw += kThreads) {
        float wv[4];
        quads.load(qw + lane, wv);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int k = 0; k < kThr; ++k) c[k] += __popcll(__ballot(wv[e] > t[k]));
      }
      __syncthreads();
      if (tid < kThr) s_above[tid] = 0;
      __syncthreads();
      if (lane == 0) {
#pragma unroll
        for (int k = 0; k < kThr; ++k)
          if (c[k]) atomicAdd(&s_above[k], c[k]);
      }
      __syncthreads();
      long long s = P.base;
#pragma unroll
      for (int k = 0; k < kThr; ++k) s += P.gain(k, s_above[k]);
      S.take(P.verdict(s), lam);
    }
  }
  if (tid == 0) {
    st.fill = -1;
    st.s = S;
    report(a, item, true, S);
  }
}

// the bit map and the tier counts, one block of units per workgroup of 256
__global__ __launch_bounds__(256) void write_kernel(MultiArgs m) {
  __shared__ int4 s_cnt[4];
  const Batched<SearchArgs>& a = m.a;
  const int row = blockIdx.y, item = a.item_of(row);
  const ItemOf it(a.batch, item);
  const int U = it.T;
  const int u0 = blockIdx.x * kBlockUnits, tid = threadIdx.x;
  if (u0 >= U) return;
  const SearchState& st = m.state[row];
  const float* __restrict__ w = a.w + it.off;
  uint8_t* __restrict__ bits = a.bits + it.off;
  float v[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] = u0 + 256 * j + tid < U ? w[u0 + 256 * j + tid] : 0.f;
  const Problem P(a, U, it.budget);
  const int n = min(kBlockUnits, U - u0);
  const int fill = st.fill >= 0 ? st.fill : (st.s.have ? -1 : P.tiers[0]);
  if (fill >= 0) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (u0 + 256 * j + tid < U) bits[u0 + 256 * j + tid] = static_cast<uint8_t>(fill);
    if (a.blk_counts && tid == 0)
      a.blk_counts[it.blk0 + blockIdx.x] =
          make_int4(fill == 16 ? n : 0, fill == 8 ? n : 0, fill == 4 ? n : 0, fill == 2 ? n : 0);
    return;
  }
  float t[kThr];
#pragma unroll
  for (int k = 0; k < kThr; ++k) t[k] = P.thr(st.s.best, k);
  int c[kThr] = {0, 0, 0, 0};
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    int above[kThr];
    const int b = tier_of(P, v[j], t, above);
    if (u0 + 256 * j + tid < U) bits[u0 + 256 * j + tid] = static_cast<uint8_t>(b);
#pragma unroll
    for (int k = 0; k < kThr; ++k) c[k] += above[k];
  }
  if (!a.blk_counts) return;
  if ((tid & 63) == 0) s_cnt[tid >> 6] = make_int4(c[0], c[1], c[2], c[3]);
  __syncthreads();
  if (tid == 0) {
    int4 x = s_cnt[0];
#pragma unroll
    for (int i = 1; i < 4; ++i) { x.x += s_cnt[i].x; x.y += s_cnt[i].y; x.z += s_cnt[i].z; x.w += s_cnt[i].w; }
    a.blk_counts[it.blk0 + blockIdx.x] = tier_counts(P, n, x);
  }
}

// Stage 3 of Alg. 1: the K budget r_K * B_head of an item is spread over its retained tokens (bit-width above zero)
// only: k_avg = min(16, 2 r_K avg_bits T / n_kept) average bits per channel unit, 0 if nothing is retained; rounded
// to fp32 like every budget.  fp64 in this operation order (the file is compiled without contraction).  The map over
// the item's 128 channels is then searched by one wavefront, two channels per lane.
struct ChannelArgs {
  AllocArgs a;                 // w, bits: the channel weights and map [items][128]
  const int4* blk_counts;      // [blocks] of the token maps: kept tokens per tier
  double rk;
};
__global__ __launch_bounds__(64) void channel_allocate_kernel(ChannelArgs c) {
  const AllocArgs& a = c.a;
  const int item = blockIdx.x, lane = threadIdx.x;
  const float* w = a.w + static_cast<int64_t>(item) * kHeadDim;
  const float v[2] = {w[lane], w[64 + lane]};
  const ItemOf it(a.batch, item);
  const int4* bc = c.blk_counts + it.blk0;
  const int nblk = (it.T + kBlockUnits - 1) / kBlockUnits;
  int kept = 0;
  for (int i = lane; i < nblk; i += 64) {
    const int4 n = bc[i];
    kept += n.x + n.y + n.z + n.w;
  }
  for (int o = 32; o > 0; o >>= 1) kept += __shfl_xor(kept, o);
  double k_avg = 0.0;
  if (kept > 0)
    k_avg = fmin(16.0, 2.0 * c.rk * it.avg * static_cast<double>(it.T) / static_cast<double>(kept));
  const Problem P(a, kHeadDim, static_cast<double>(static_cast<float>(k_avg)));
  uint8_t* bits = a.bits + static_cast<int64_t>(item) * kHeadDim;
  const int fill = P.fill(kHeadDim);
  Search S{0.0, 0.0, 0.0, 0, 0, 0};
  float t[kThr];
  if (fill < 0) {
    S.hi = static_cast<double>(wave_max(fmaxf(fmaxf(v[0], v[1]), 0.f)));
    steps_in_wave<2>(P, v, P.base, bracket_of(S), S);
#pragma unroll
    for (int k = 0; k < kThr; ++k) t[k] = S.have ? P.thr(S.best, k) : INFINITY;
  }
  int tier[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    int above[kThr];
    tier[j] = fill >= 0 ? fill : tier_of(P, v[j], t, above);
    bits[64 * j + lane] = static_cast<uint8_t>(tier[j]);
  }
  if (a.post.channels) {                   // word 4 k + p: which of the channels 32 p .. 32 p + 31 have 16 >> k bits
    uint32_t word = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const uint64_t mask = __ballot(tier[j] == 16 >> k);
        if (lane >> 1 == 2 * k + j) word = static_cast<uint32_t>(lane & 1 ? mask >> 32 : mask);
      }
    if (lane < 16) post_word(a.post.channels, 16 * static_cast<int64_t>(item) + lane, a.post.tag, word);
  }
  if (lane == 0) report(a, item, fill < 0, S);
}

AllocArgs make_args(const float* w, const Batch& batch, int n_hull, const int* hull_tiers, const double* hull_r, double need_frac,
                    int max_iters, uint8_t* bits, double* lam_out, int32_t* iters_out) {
  AllocArgs a{};
  a.w = w; a.bits = bits; a.batch = batch;
  for (int k = 0; k < kMaxHull; ++k) {
    a.tiers[k] = k < n_hull ? hull_tiers[k] : 0;
    a.r[k] = k < n_hull - 1 ? hull_r[k] : 0.0;
  }
  a.n_hull = n_hull; a.max_iters = max_iters; a.need_frac = need_frac;
  a.lam_out = lam_out; a.iters_out = iters_out;
  return a;
}

size_t hist_bytes(int n_items) { return static_cast<size_t>(n_items) * Anchored::kBuckets * sizeof(int32_t); }
size_t state_bytes(int n_items) { return (static_cast<size_t>(n_items) * sizeof(SearchState) + 255) / 256 * 256; }

// Items that the many-workgroup form takes at once: 130 KB of scratch each, 67 MB in all.
constexpr int kMostTogether = 512;

hipError_t launch_short_items(AllocArgs a, int n_items, int max_U, hipStream_t st) {
  // The launch ends with its slowest item, and of many some have more steps left than the list is worth: 32 items of 12K units
  // 23.9 -> 22.4 us with up to nine such steps, 64 of 11K 26.8 -> 22.5, 128 of 14K 27.4 -> 28.9.
  a.direct = n_items <= 64 ? 9 : 0;
  const dim3 grid(n_items), block(kThreads);
#define RDKV_ITEMS(REG_)                                                              \
  {                                                                                   \
    const hipError_t e = RDKV_ALLOW_LDS((allocate_item_kernel<REG_>), kItemLds<REG_>); \
    if (e != hipSuccess) return e;                                                    \
    hipLaunchKernelGGL(allocate_item_kernel<REG_>, grid, block, kItemLds<REG_>, st, a); \
  }
  if (max_U <= 4 * kThreads) RDKV_ITEMS(4)
  else if (max_U <= 8 * kThreads) RDKV_ITEMS(8)
  else if (max_U <= 16 * kThreads) RDKV_ITEMS(16)
  else RDKV_ITEMS(32)
#undef RDKV_ITEMS
  return hipGetLastError();
}

hipError_t launch_items_together(const AllocArgs& a, int n_items, int max_U, void* scratch, hipStream_t st) {
  MultiArgs m;
  static_cast<SearchArgs&>(m.a) = a;
  m.a.order = a.order; m.a.batch = a.batch;
  uint8_t* p = static_cast<uint8_t*>(scratch);
  m.hist = reinterpret_cast<int32_t*>(p);
  m.state = reinterpret_cast<SearchState*>(p + hist_bytes(n_items));
  m.list = reinterpret_cast<float*>(p + hist_bytes(n_items) + state_bytes(n_items));
  m.slice_max = m.list + static_cast<size_t>(n_items) * kListCap;
  m.slices = std::max(1, std::min(kMostSlices, 256 / n_items));
  m.maxima = std::max(1, std::min(kMostMaxima, 512 / n_items));
  const int64_t clear = static_cast<int64_t>((hist_bytes(n_items) + state_bytes(n_items)) / 16);
  const dim3 wide(m.slices, n_items), block(kThreads);
  const dim3 first(m.maxima, n_items);
  if (a.raw) hipLaunchKernelGGL(slice_max_kernel<true>, first, block, 0, st, m, const_cast<float*>(a.w), reinterpret_cast<uint4*>(p), clear);
  else hipLaunchKernelGGL(slice_max_kernel<false>, first, block, 0, st, m, nullptr, reinterpret_cast<uint4*>(p), clear);
  hipError_t e = RDKV_ALLOW_LDS(hist_kernel, kHistLds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(hist_kernel, wide, block, kHistLds, st, m);
  e = RDKV_ALLOW_LDS(gather_kernel, kGatherLds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(gather_kernel, wide, block, kGatherLds, st, m);
  hipLaunchKernelGGL(write_kernel, dim3((max_U + kBlockUnits - 1) / kBlockUnits, n_items), dim3(256), 0, st, m);
  return hipGetLastError();
}

}  // namespace

// How a batch is searched.  Up to 32K units per item: one launch, a workgroup per item.  Longer ones and up to 512 items:
// all of them in the many-workgroup form (8 items of 128K units and 8 of 20K: 38 us).  More items: those beyond 32K units in
// groups of 512, so that the scratch has a bound, and the others in the launch of their own.
bool allocate_needs_order(int n_items, int max_U) { return max_U > kItemUnits && n_items > kMostTogether; }
int allocate_short_units() { return kItemUnits; }

// Device scratch launch_allocate needs for items of up to max_U units; 0 where one workgroup holds an item.
size_t allocate_scratch_bytes(int n_items, int max_U) {
  if (max_U <= kItemUnits) return 0;
  const int n = std::min(n_items, kMostTogether);
  return hist_bytes(n) + state_bytes(n) + static_cast<size_t>(n) * (kListCap + kMostMaxima) * sizeof(float);
}

// Token maps of all items.  d_order (where allocate_needs_order): the items, the n_long of more than allocate_short_units()
// first, the others with up to max_short units.  blk_counts: what the packing stage needs, or null.
// post: where the items' counts go for the host, which only the launch of whole items does (up to allocate_short_units units).
// raw: the weights before the pooling (window pool > 1), which the search then does itself; w is memory for the pooled ones.
hipError_t launch_allocate(const float* raw, int pool, float* w, const Batch& batch, int max_U, const int32_t* d_order, int n_long,
                           int max_short, int n_hull, const int* hull_tiers,
                           const double* hull_r, double need_frac, int max_iters, uint8_t* bits, double* lam_out,
                           int32_t* iters_out, int32_t* blk_counts, const CountPost& post, void* scratch, hipStream_t st) {
  const int n_items = batch.n_seqs * batch.hkv;
  if (n_items == 0) return hipSuccess;
  if (n_hull < 1 || n_hull > kMaxHull) return hipErrorInvalidValue;
  AllocArgs a = make_args(w, batch, n_hull, hull_tiers, hull_r, need_frac, max_iters, bits, lam_out, iters_out);
  a.blk_counts = reinterpret_cast<int4*>(blk_counts);
  if (pool > 1) {
    a.raw = raw;
    a.pool = pool;
    a.pool_inv = 1.0f / static_cast<float>(pool);
  }
  if (max_U <= kItemUnits) {
    if (a.blk_counts) a.post = post;
    return launch_short_items(a, n_items, max_U, st);
  }
  if (!scratch || (!d_order && n_items > kMostTogether)) return hipErrorInvalidValue;
  if (!d_order) return launch_items_together(a, n_items, max_U, scratch, st);
  for (int first = 0; first < n_long; first += kMostTogether) {
    a.order = d_order + first;
    const hipError_t e = launch_items_together(a, std::min(kMostTogether, n_long - first), max_U, scratch, st);
    if (e != hipSuccess) return e;
  }
  a.order = d_order + n_long;
  return n_items > n_long ? launch_short_items(a, n_items - n_long, max_short, st) : hipSuccess;
}

// Stage 3: the channel maps, from the kept tokens launch_allocate has counted.
hipError_t launch_allocate_channels(const float* w_ch, const Batch& batch, const int32_t* blk_counts, double rk, int n_hull,
                                    const int* hull_tiers,
                                    const double* hull_r, double need_frac, int max_iters, uint8_t* bits_ch,
                                    double* lam_out, int32_t* iters_out, const CountPost& post, hipStream_t st) {
  const int n_items = batch.n_seqs * batch.hkv;
  if (n_items == 0) return hipSuccess;
  if (n_hull < 1 || n_hull > kMaxHull) return hipErrorInvalidValue;
  ChannelArgs c;
  c.a = make_args(w_ch, batch, n_hull, hull_tiers, hull_r, need_frac, max_iters, bits_ch, lam_out, iters_out);
  c.blk_counts = reinterpret_cast<const int4*>(blk_counts); c.rk = rk;
  c.a.post = post;
  hipLaunchKernelGGL(channel_allocate_kernel, dim3(n_items), dim3(64), 0, st, c);
  return hipGetLastError();
}

}  // namespace rdkv
