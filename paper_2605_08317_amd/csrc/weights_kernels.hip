// Stage 1 of Alg. 1 on the GPU: token weights (Eq. 2) and channel weights (Eq. 4).
//
// The token weights need S = Q_obs K^T / sqrt(d) for the R = g * S_w window rows of
// a KV head against all T keys -- a dense [R x 128] x [128 x T] contraction, done
// with bf16 MFMA (v_mfma_f32_16x16x32_bf16) and never stored.  Two streaming
// passes over K: pass 1 produces the log-sum-exp of every row (softmax
// normaliser), pass 2 recomputes the logits and accumulates the column sums
// w_t = sum_rows exp(s - lse_row).  Pass 1 also accumulates the per-channel sum of
// squares of K for the channel weights.
//
// Both passes hold the window rows in registers (64 rows per wavefront, 256 per workgroup and sweep) and stream a run of
// keys through three LDS buffers of 64 keys, copied there without passing through registers, so that the rows are
// fetched once per run and two tiles of keys are in flight during the arithmetic on a third.  The products of a step are
// issued between the exponentials of the step before: a logit costs the plain ALUs a multiply-add, an exponential (8
// cycles per wavefront) and an addition beside the matrix core.  Measured: 8 heads x 128K keys x 256 rows 109 + 102 us
// -> 76 + 78 us for the two passes (kernel trace; 85 + 92 among other work), 128 heads x 20K keys x 256 rows 256 + 239 ->
// 179 + 184 us (keys stationary and rows staged through LDS before).  What bounds them: matrix core and plain ALUs together.
// The products alone are 69 GFLOP per pass of the first shape, 58 us at the rate a large library product reaches on this card
// (1.18 PFLOP/s; its clock drops under matrix work on random data).  By the counters two wavefronts per SIMD fill two thirds
// of the vector issue, keep the matrix core busy 53 to 55 % of their time and wait 20 to 24 % of it; keys arrive at 3.4 TB/s.
// Tile shapes, occupancy (2 or 3 wavefronts per SIMD) and deeper prefetch change nothing.
#include <algorithm>
#include <type_traits>

#include "rdkv_internal.h"
#include "wave_ops.h"
#include "weights_plan.h"

namespace rdkv {

namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;

constexpr int kKeyTileBytes = kKeyTile * kHeadDim * 2;   // an LDS buffer
constexpr int kBuffers = 3;                 // two tiles in flight while one is computed
constexpr int kSumTiles = 16;               // tiles whose column sums pass 2 keeps in LDS
constexpr int kPass1PerCu = 2, kPass2PerCu = 2;   // workgroups a compute unit keeps resident (registers)
constexpr float kNegBig = -1.0e30f;
constexpr float kLogitScale = 1.4426950408889634f * 0.08838834764831845f;   // log2(e) / sqrt(128)

struct WeightArgs {
  const uint16_t* K;
  const uint16_t* Q;             // [batch][hq][s_obs][d]
  float* row_part;               // [workgroups + items][row_slots][2]  (m, l) in the log2 domain
  float* lse;                    // [items][row_slots], or null: pass 2 makes it from the partials
  float* w_raw;                  // [total tokens] unpooled weights
  float* ksq_part;               // [workgroups + items][128] or null
  int32_t hq, hkv, g, s_obs, R, row_slots, causal;   // row_slots: R in whole sweeps of row groups
  int32_t n_items, n_tiles;      // items, key tiles of all of them
  int32_t workgroups;            // pass 1
  Batch batch;
  int32_t sum_workgroups;        // pass 2, of those that sum
  float* w_ch;                   // [items][128]: where pass 2's other workgroups leave the channel weights, or null
};

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// a table entry every lane has read alike, as a scalar
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t uniform64(int64_t v) {
  return static_cast<int64_t>(static_cast<uint32_t>(uniform(static_cast<int>(v)))) |
         (static_cast<int64_t>(uniform(static_cast<int>(v >> 32))) << 32);
}

// 16 bytes per lane from global memory straight into LDS: lane i's bytes, base + offset, land at lds_base + 16 i (base
// and lds_base are uniform).  The compiler does not see the copy, so the reader waits for it by hand (tile_barrier).
__device__ __forceinline__ void copy_to_lds(const void* base, uint32_t offset, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(offset), "s"(base), "s"(lds_base) : "memory", "m0");
}
// Barrier of the workgroup after this wavefront's vector memory operations but the last PENDING have completed.
template <int PENDING>
__device__ __forceinline__ void tile_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(PENDING) : "memory");
}

// The key tiles of all items in one line are cut into `workgroups` runs that differ by at most one tile, so that every
// workgroup of a launch that fits the chip once has the same amount of work whatever the lengths of the items.  A run
// may cover the end of one item and the start of the next; what workgroup w leaves about item i goes to slot w + i,
// which no other pair has, and an item's slots are consecutive.
__device__ __forceinline__ int first_tile(int w, int workgroups, int n_tiles) {
  return static_cast<int>(static_cast<int64_t>(w) * n_tiles / workgroups);
}
__device__ __forceinline__ int owner_of(int tile, int workgroups, int n_tiles) {   // largest w with first_tile(w) <= tile
  return static_cast<int>(((static_cast<int64_t>(tile) + 1) * workgroups + n_tiles - 1) / n_tiles) - 1;
}
// slots of an item: [*first, *first + return value)
__device__ __forceinline__ int item_slots(const WeightArgs& a, int item, int* first) {
  const ItemOf it(a.batch, item);
  const int t0 = it.tile0, t1 = t0 + it.tiles();
  *first = 0;
  if (t1 <= t0) return 0;
  const int w0 = owner_of(t0, a.workgroups, a.n_tiles), w1 = owner_of(t1 - 1, a.workgroups, a.n_tiles);
  *first = w0 + item;
  return w1 - w0 + 1;
}

// The log-sum-exp (log2 domain) of a row of an item of n <= MANY runs (p: the first one's), with the additions of
// row_lse_kernel, whose sixteen threads have at most three runs each then.
template <int MANY>
__device__ __forceinline__ float lse_of_few(const float2* p, int row_slots, int n) {
  static_assert(MANY <= 48, "three runs a thread");
  float2 v[MANY];
#pragma unroll
  for (int k = 0; k < MANY; ++k) v[k] = p[static_cast<int64_t>(min(k, n - 1)) * row_slots];     // (the last one repeated, without a branch)
  float m = kNegBig, l = 0.f;
#pragma unroll
  for (int k = 0; k < MANY; ++k) m = fmaxf(m, v[k].x);
#pragma unroll
  for (int k = 0; k < min(MANY, 16); ++k) {
    float own = v[k].x, sum = k < n ? v[k].y : 0.f;
    if (k + 16 < MANY) {
      const float2 hi = v[(k + 16) % MANY], top = v[(k + 32) % MANY];
      const bool third = k + 32 < MANY && k + 32 < n;
      own = k + 16 < n ? fmaxf(own, hi.x) : own;
      if (k + 32 < MANY) own = third ? fmaxf(own, top.x) : own;
      sum = sum * fast_exp2(v[k].x - own) + (k + 16 < n ? hi.y * fast_exp2(hi.x - own) : 0.f);
      if (k + 32 < MANY) sum += third ? top.y * fast_exp2(top.x - own) : 0.f;
    }
    l += sum * fast_exp2(own - m);
  }
  return l > 0.f ? m + __log2f(l) : INFINITY;
}

// w_c = ||Q[:,c]|| ||K[:,c]|| / sqrt(d): finishes the K sums of squares and adds the probe's column norms; a workgroup has
// kChannelPart channels of an item, 8 threads per channel share the runs and the window rows (fixed order of additions).
// Part of row_lse_kernel's launch, or of pass 2's where it makes the log-sum-exp itself: all need what pass 1 leaves (as a launch of
// its own 4 us of a pass over 8 x 50K keys).
constexpr int kChannelPart = 32;
__device__ __forceinline__ void channel_weights(const WeightArgs& a, float* __restrict__ w_ch, int item, int part) {
  static_assert(8 * kChannelPart == 256, "the threads of the kernels");
  __shared__ float s_k[8][kChannelPart], s_q[8][kChannelPart];
  const int lc = threadIdx.x & (kChannelPart - 1), sub = threadIdx.x / kChannelPart;
  const int c = part * kChannelPart + lc;
  int slot0;
  const int n = item_slots(a, item, &slot0);
  const int64_t b0 = slot0;
  float ksq = 0.f;
#pragma unroll 8
  for (int b = sub; b < n; b += 8) ksq += a.ksq_part[(b0 + b) * kHeadDim + c];
  const int seq = item / a.hkv, head = item % a.hkv;
  const uint16_t* Qg = a.Q + (static_cast<int64_t>(seq) * a.hq + head * a.g) * a.s_obs * kHeadDim;
  float qsq = 0.f;
#pragma unroll 8
  for (int r = sub; r < a.R; r += 8) {
    const float q = __uint_as_float(static_cast<uint32_t>(Qg[r * kHeadDim + c]) << 16);
    qsq = __builtin_fmaf(q, q, qsq);
  }
  s_k[sub][lc] = ksq;
  s_q[sub][lc] = qsq;
  __syncthreads();
  if (sub == 0) {
    ksq = qsq = 0.f;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      ksq += s_k[k][lc];
      qsq += s_q[k][lc];
    }
    w_ch[static_cast<int64_t>(item) * kHeadDim + c] = sqrtf(qsq) * sqrtf(ksq) * 0.08838834764831845f;
  }
}

// One workgroup = one run of key tiles against all window rows of their items.
//   NRT  32-row tiles of window rows per wavefront: 2, or 1 when the item has at most 64 rows
//   RGW  row groups (of 32 NRT rows) worked on at a time: 4, or 2 when the item has at most 128 rows
//   KSQ  pass 1 also sums the squares of K per channel; pass 2 has workgroups behind the others that finish the channel weights
// A wavefront owns row group wave % RGW and, of the two 32-key steps of a tile, both (RGW = 4) or one; more than four
// row groups take a second sweep over the run.
// The LDS image of a key tile is row-major with the 16-byte pieces of key r at position piece ^ (r % 16), which spreads
// keys that are read at one column over all banks.
// Products on v_mfma_f32_32x32x16_bf16: a product of the 16x16x32 shape takes as many issue cycles from the plain ALUs
// (eight, measured) and does half the work.  Result register r of lane (half, l32) holds element 8 (r / 4) + 4 half + r % 4
// of the A side against element l32 of the B side:
//   pass 1: A = keys, B = rows: a lane has one window row and 16 keys of the step
//   pass 2: A = rows, B = keys: a lane has one key and 16 rows of the row tile
template <int PASS, int NRT, int RGW, bool KSQ>
__global__ __launch_bounds__(256, PASS == 1 ? kPass1PerCu : kPass2PerCu) void weights_kernel(WeightArgs a) {
  __shared__ __align__(16) uint8_t s_keys[kBuffers][kKeyTileBytes];
  __shared__ float s_sum[PASS == 2 ? kSumTiles : 1][RGW][PASS == 2 ? kKeyTile : 1];   // pass 2: [tile % kSumTiles][row group][key]

  constexpr int kRows = RGW * 32 * NRT;                // of a sweep
  float* s_lse = &s_sum[0][0][0];                      // [kRows], before the first column sums

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5;
  const int n_groups = (a.R + 32 * NRT - 1) / (32 * NRT);
  constexpr int kSplit = 4 / RGW;                      // wavefronts that share a row group
  constexpr int kSteps = 2 / kSplit;                   // 32-key steps of a tile per wavefront
  const int rgi = wave % RGW, ks = wave / RGW;
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(&s_keys[0][0]));   // LDS byte address
  const int prow = tid >> 4, piece = (tid & 15) ^ (prow & 15);   // this thread's key rows prow + 16 k and piece of the key

  constexpr bool kSquares = PASS == 1 && KSQ;
  int workgroups = gridDim.x;
  if constexpr (PASS == 2 && KSQ) {
    workgroups = a.sum_workgroups;
    if (static_cast<int>(blockIdx.x) >= workgroups) {
      constexpr int kParts = kHeadDim / kChannelPart;
      const int k = static_cast<int>(blockIdx.x) - workgroups;
      channel_weights(a, a.w_ch, k / kParts, k % kParts);
      return;
    }
  }
  const int run0 = first_tile(blockIdx.x, workgroups, a.n_tiles), run1 = first_tile(blockIdx.x + 1, workgroups, a.n_tiles);
  int seq = 0;                             // the sequence of tile run0: the last one that starts at or before it
  for (int s0 = 0; s0 < a.batch.n_seqs && a.batch.n_seqs > 1; s0 += 64) {
    const int s = s0 + lane;
    const uint64_t before = __ballot(s < a.batch.n_seqs && a.batch.tile0(min(s, a.batch.n_seqs - 1)) <= run0);
    if (before == 0) break;
    seq = s0 + 63 - __clzll(static_cast<long long>(before));
  }
  int head = -1;                           // (not known yet)
  for (int tile0 = run0; tile0 < run1; ++head) {
  if (head == a.hkv) {
    head = 0;
    ++seq;
  }
  const SeqEntry entry = a.batch.seq(seq);
  const int T = uniform(entry.T), tiles = (T + kKeyTile - 1) / kKeyTile;
  if (head < 0) head = (tile0 - uniform(entry.tile0)) / tiles;      // (the sequence has the tile, so it has keys)
  const int item = seq * a.hkv + head, item0 = uniform(entry.tile0) + head * tiles;
  const int ntile = min(run1, item0 + tiles) - tile0;   // this run's tiles of the item
  if (ntile <= 0) continue;                // an item without keys
  const int64_t row_off = uniform64(entry.row0) + static_cast<int64_t>(head) * T;
  const int key0 = (tile0 - item0) * kKeyTile, key1 = min(T, key0 + ntile * kKeyTile);
  tile0 += ntile;
  const int per_s_obs = 65536 / a.s_obs + 1;
  const uint16_t* Qg = a.Q + (static_cast<int64_t>(seq) * a.hq + head * a.g) * a.s_obs * kHeadDim;
  const uint16_t* Kh = a.K + row_off * kHeadDim;
  const int64_t blk = static_cast<int64_t>(blockIdx.x) + item;
  // leading tiles of 64 valid keys that every row may look at (keys up to T - s_obs)
  const int n_plain = max(0, min(key1, a.causal ? T - a.s_obs + 1 : T) - key0) / kKeyTile;
  float ksq[8];
  if constexpr (kSquares) {
#pragma unroll
    for (int j = 0; j < 8; ++j) ksq[j] = 0.f;
  }

  for (int sweep = 0; sweep * RGW < n_groups; ++sweep) {
    const int row0 = (sweep * RGW + rgi) * 32 * NRT;   // first window row of this wavefront
    // Tiles past the run's last are fetched too (its last tile once more, into a buffer nobody reads), so that the
    // number of copies in flight does not depend on the tile.
    const auto fetch = [&](int t, int buffer) __attribute__((always_inline)) {
      const uint32_t base = lds0 + static_cast<uint32_t>(buffer) * kKeyTileBytes + wave * 1024;
      const int first = key0 + min(t, ntile - 1) * kKeyTile, last = T - 1 - first;
      const uint16_t* src = Kh + static_cast<int64_t>(first) * kHeadDim;
#pragma unroll
      for (int k = 0; k < 4; ++k)
        copy_to_lds(src, static_cast<uint32_t>(min(prow + 16 * k, last) * (kHeadDim * 2) + piece * 16), base + 4096 * k);
    };
    int cur = 0;                           // buffer of the next tile to be opened
    const auto start = [&]() __attribute__((always_inline)) {
      cur = 0;
#pragma unroll
      for (int t = 0; t < kBuffers - 1; ++t) fetch(t, t);
    };
    // Tile t's keys: this wavefront's part has landed (kBuffers - 2 younger tiles may be in flight), and after the
    // barrier everybody's has; the buffer of tile t - 1 is free then and takes tile t + kBuffers - 1.
    const auto open_tile = [&](int t, bool squares) __attribute__((always_inline)) -> const uint8_t* {
      tile_barrier<4 * (kBuffers - 2)>();
      fetch(t + kBuffers - 1, cur == 0 ? kBuffers - 1 : cur - 1);
      const uint8_t* buf = s_keys[cur];
      cur = cur + 1 == kBuffers ? 0 : cur + 1;
      if constexpr (kSquares) {
        if (squares && sweep == 0) {
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const uint4 v = *reinterpret_cast<const uint4*>(buf + (prow + 16 * k) * (kHeadDim * 2) + (tid & 15) * 16);
            if (key0 + t * kKeyTile + prow + 16 * k < key1) {
              const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
              for (int j = 0; j < 4; ++j) {
                const float lo = __uint_as_float(w[j] << 16), hi = __uint_as_float(w[j] & 0xFFFF0000u);
                ksq[2 * j] = __builtin_fmaf(lo, lo, ksq[2 * j]);
                ksq[2 * j + 1] = __builtin_fmaf(hi, hi, ksq[2 * j + 1]);
              }
            }
          }
        }
      }
      return buf;
    };
    start();
    if constexpr (PASS == 2) {
      if (a.lse == nullptr) {              // while the first keys arrive; n_tiles workgroups stays below 2^32
        const uint32_t tiles_end = static_cast<uint32_t>(item0 + (lane == 0 ? 1 : tiles)) * static_cast<uint32_t>(a.workgroups);
        const int w = static_cast<int>((tiles_end + static_cast<uint32_t>(a.n_tiles) - 1) / static_cast<uint32_t>(a.n_tiles)) - 1;   // owner_of the item's first tile, its last
        const int w0 = uniform(w), n = __builtin_amdgcn_readlane(w, 1) - w0 + 1;
        const int row = sweep * kRows + tid;
        const float2* p = reinterpret_cast<const float2*>(a.row_part) + static_cast<int64_t>(w0 + item) * a.row_slots + row;
        if (tid < kRows) s_lse[tid] = row >= a.R ? INFINITY : n <= 8 ? lse_of_few<8>(p, a.row_slots, n) : lse_of_few<kFewRuns>(p, a.row_slots, n);
        __syncthreads();
      }
    }
    // window rows past the last repeat it: pass 1 drops their sums, pass 2 gives them a log-sum-exp of infinity
    bf16x8 q_op[NRT][8];
#pragma unroll
    for (int rt = 0; rt < NRT; ++rt) {
      const uint16_t* qrow = Qg + static_cast<int64_t>(min(row0 + rt * 32 + l32, a.R - 1)) * kHeadDim + half * 8;
#pragma unroll
      for (int kb = 0; kb < 8; ++kb) q_op[rt][kb] = *reinterpret_cast<const bf16x8*>(qrow + kb * 16);
    }
    float m[NRT], l[NRT];                  // pass 1: reference and sum of this lane's keys for its row of each tile
    float nlse[PASS == 2 ? NRT : 1][16];   // pass 2: minus the log-sum-exp of this lane's rows
    if constexpr (PASS == 1) {
#pragma unroll
      for (int rt = 0; rt < NRT; ++rt) { m[rt] = kNegBig; l[rt] = 0.f; }
    } else {
#pragma unroll
      for (int rt = 0; rt < NRT; ++rt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int r = (rgi * NRT + rt) * 32 + 8 * i + 4 * half;
          float4 v;
          if (a.lse) v = *reinterpret_cast<const float4*>(a.lse + static_cast<int64_t>(item) * a.row_slots + sweep * kRows + r);
          else v = *reinterpret_cast<const float4*>(s_lse + r);
          nlse[rt][4 * i] = -v.x; nlse[rt][4 * i + 1] = -v.y; nlse[rt][4 * i + 2] = -v.z; nlse[rt][4 * i + 3] = -v.w;
        }
    }

    // piece kb (16 channels) of the keys of one 32-key step, as an operand
    const auto read_keys = [&](const uint8_t* buf, int step, int kb) __attribute__((always_inline)) {
      return *reinterpret_cast<const bf16x8*>(buf + (step * 32 + l32) * (kHeadDim * 2) + (((kb * 2 + half) ^ (l32 & 15)) * 16));
    };
    const auto product = [&](bf16x8 k, int rt, int kb, floatx16 c) __attribute__((always_inline)) {
      return PASS == 1 ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(k, q_op[rt][kb], c, 0, 0, 0)
                       : __builtin_amdgcn_mfma_f32_32x32x16_bf16(q_op[rt][kb], k, c, 0, 0, 0);
    };
    constexpr floatx16 kZero = {};
    bf16x8 k_op[8];
    const auto logits = [&](int rt) __attribute__((always_inline)) {
      floatx16 c = kZero;
#pragma unroll
      for (int kb = 0; kb < 8; ++kb) c = product(k_op[kb], rt, kb, c);
      return c;
    };
    const auto element = [&](int r) { return 8 * (r >> 2) + 4 * half + (r & 3); };   // A-side element of result register r
    // last key row `row` of the window may look at
    // (row % s_obs by a product: rows stay below 768 and s_obs is at most 64, where 65536 / s_obs + 1 is exact enough.  The
    // division, 32 of them per lane and step, made the workgroups with an item's last tile 5 us slower than the others.)
    const auto limit_of = [&](int row) {
      const int i = row - static_cast<int>((static_cast<uint32_t>(row) * static_cast<uint32_t>(per_s_obs)) >> 16) * a.s_obs;
      return min(a.causal ? T - a.s_obs + i : T - 1, key1 - 1);
    };

    // One position of the pipeline over the plain tiles (a position = a step against one row tile): the products of a
    // position, whose keys are in k_op, issued one by one between the exponentials of the position before (acc), and,
    // in a step's last position, k_op refilled with the next step (a piece as soon as its product is issued).
    floatx16 acc;
    float part[4];                          // pass 2: column sums of the step under way
    const auto position = [&](auto multiply, auto mul_rt, auto done_rt, const uint8_t* rbuf, int rstep, int t,
                              int step) __attribute__((always_inline)) {
      constexpr bool kMultiply = decltype(multiply)::value;
      constexpr int kMulRt = decltype(mul_rt)::value, kRt = decltype(done_rt)::value;
      floatx16 nxt;
      float x[2][2], e[2] = {0.f, 0.f}, sum = 0.f;
      const auto scaled = [&](int p) __attribute__((always_inline)) {
        return __builtin_fmaf(acc[p], kLogitScale, PASS == 1 ? -m[kRt] : nlse[PASS == 2 ? kRt : 0][p]);
      };
      // Pass 1: the reference m is a logit this lane has seen and stays what it is: fp32 carries sums up to 2^100 times
      // its exponential, and a run that exceeds that is done again with a running maximum.
      const auto add = [&](int p, float v) __attribute__((always_inline)) {
        if constexpr (PASS == 1) sum = p == 0 ? v : sum + v;
        else part[p & 3] = kRt == 0 && p < 4 ? v : part[p & 3] + v;
      };
      x[0][0] = scaled(0);
      x[0][1] = scaled(1);
#pragma unroll
      for (int kb = 0; kb < 8; ++kb) {      // logits 2 kb and 2 kb + 1 of the finished position
        if constexpr (kMultiply) {
          nxt = product(k_op[kb], kMulRt, kb, kb == 0 ? kZero : nxt);
          if (kMulRt == NRT - 1) k_op[kb] = read_keys(rbuf, rstep, kb);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          if (kb < 7) x[(kb + 1) & 1][u] = scaled(2 * kb + 2 + u);
          const float en = fast_exp2(x[kb & 1][u]);
          if (kb > 0) add(2 * kb - 2 + u, e[u]);
          e[u] = en;
        }
        if constexpr (kMultiply) __builtin_amdgcn_sched_barrier(0);
      }
      add(14, e[0]);
      add(15, e[1]);
      if constexpr (PASS == 1) {
        l[kRt] += sum;
      } else if constexpr (kRt == NRT - 1) {
        const float own = (part[0] + part[1]) + (part[2] + part[3]), c = halves_sum(own, own);
        if (half == 0) s_sum[t % kSumTiles][rgi][step * 32 + l32] = c;
      }
      if constexpr (kMultiply) acc = nxt;
    };
    // Pass 2: the column sums of tiles t0 .. t1 - 1, whose steps are behind a barrier, added over the row groups.  Eight
    // tiles at a time: a store holds back the wait for the next tile's keys until it is acknowledged.
    const auto flush = [&](int t0, int t1) __attribute__((always_inline)) {
      if constexpr (PASS == 2) {
        for (int i = tid; i < (t1 - t0) * kKeyTile; i += 256) {
          const int t = t0 + (i >> 6), key = key0 + t0 * kKeyTile + i;
          if (key < key1) {
            float s = 0.f;
#pragma unroll
            for (int k = 0; k < RGW; ++k) s += s_sum[t % kSumTiles][k][i & 63];
            float* dst = a.w_raw + row_off + key;
            *dst = sweep == 0 ? s : *dst + s;
          }
        }
      }
    };
    // after opening tile t + 1 (t + 2 where a tile is one position): tiles up to t - 1 are complete
    const auto flush_some = [&](int t) __attribute__((always_inline)) {
      if (PASS == 2 && t > 0 && t % (kSumTiles / 2) == 0) flush(t - kSumTiles / 2, t);
    };

    // ---- plain tiles -----------------------------------------------------------------------------------------------
    if (n_plain > 0) {
      using std::integral_constant;
      using std::false_type;
      using std::true_type;
      constexpr int kPos = kSteps * NRT;    // positions of a tile
      constexpr integral_constant<int, 0> first_rt{};
      constexpr integral_constant<int, NRT - 1> last_rt{};
      const uint8_t* buf = open_tile(0, true);
#pragma unroll
      for (int kb = 0; kb < 8; ++kb) k_op[kb] = read_keys(buf, ks, kb);
#pragma unroll
      for (int rt = NRT - 1; rt >= 0; --rt) {   // position 0; the other row tiles' references in pass 1
        if (PASS == 2 && rt > 0) continue;
        acc = logits(rt);
        if constexpr (PASS == 1) {
          float mx = acc[0];
#pragma unroll
          for (int r = 1; r < 16; ++r) mx = fmaxf(mx, acc[r]);
          m[rt] = mx * kLogitScale;
        }
      }
      if constexpr (kPos == 1) {
        if (n_plain > 1) buf = open_tile(1, true);
#pragma unroll
        for (int kb = 0; kb < 8; ++kb) k_op[kb] = read_keys(buf, ks, kb);
      }
      // position j of tile t multiplies position j (position 0 of the next tile for j = kPos) and finishes position
      // j - 1; a tile is opened in the position that fetches its first step
      for (int t = 0; t + 1 < n_plain; ++t) {
        if constexpr (kPos == 1) {
          if (t + 2 < n_plain) {
            buf = open_tile(t + 2, true);
            flush_some(t);
          }
          position(true_type{}, first_rt, first_rt, buf, ks, t, ks);
        } else {
          if constexpr (kPos == 4) {
            position(true_type{}, last_rt, first_rt, buf, ks + kSplit, t, ks);
            position(true_type{}, first_rt, last_rt, buf, 0, t, ks);
          }
          buf = open_tile(t + 1, true);
          flush_some(t);
          position(true_type{}, last_rt, first_rt, buf, ks, t, ks + (kSteps - 1) * kSplit);
          position(true_type{}, first_rt, last_rt, buf, 0, t, ks + (kSteps - 1) * kSplit);
        }
      }
      if constexpr (kPos == 4) {
        position(true_type{}, last_rt, first_rt, buf, ks + kSplit, n_plain - 1, ks);
        position(true_type{}, first_rt, last_rt, buf, 0, n_plain - 1, ks);
      }
      if constexpr (kPos > 1) position(true_type{}, last_rt, first_rt, buf, ks, n_plain - 1, ks + (kSteps - 1) * kSplit);
      position(false_type{}, first_rt, last_rt, buf, 0, n_plain - 1, ks + (kSteps - 1) * kSplit);
      if constexpr (PASS == 2) {
        __syncthreads();
        // what flush_some has left (the last t it was called with is n_plain - 2, or n_plain - 3)
        flush(max(0, n_plain - (kPos == 1 ? 3 : 2)) / (kSumTiles / 2) * (kSumTiles / 2), n_plain);
      }
    }

    // ---- the run's other tiles: masks, and in pass 1 a running maximum --------------------------------------------
    int t0 = n_plain;
    if constexpr (PASS == 1) {
      bool fits = true;
#pragma unroll
      for (int rt = 0; rt < NRT; ++rt) fits = fits && l[rt] < 1.0e30f;
      if (n_plain > 0 && !__syncthreads_and(fits)) {   // logits further apart than fp32 carries: all over again
        t0 = 0;
        tile_barrier<0>();
        start();
#pragma unroll
        for (int rt = 0; rt < NRT; ++rt) { m[rt] = kNegBig; l[rt] = 0.f; }
      }
    }
    for (int t = t0; t < ntile; ++t) {
      const uint8_t* buf = open_tile(t, t >= n_plain);
#pragma unroll 1
      for (int step = ks; step < 2; step += kSplit) {
#pragma unroll
        for (int kb = 0; kb < 8; ++kb) k_op[kb] = read_keys(buf, step, kb);
        const int step0 = key0 + t * kKeyTile + step * 32;
        float c = 0.f;
#pragma unroll
        for (int rt = 0; rt < NRT; ++rt) {
          acc = logits(rt);
          if constexpr (PASS == 1) {
            const int limit = limit_of(row0 + rt * 32 + l32);
            float mx = m[rt];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              acc[r] = step0 + element(r) <= limit ? acc[r] * kLogitScale : -INFINITY;
              mx = fmaxf(mx, acc[r]);
            }
            float s = l[rt] * fast_exp2(m[rt] - mx);
#pragma unroll
            for (int r = 0; r < 16; ++r) s += fast_exp2(acc[r] - mx);
            m[rt] = mx;
            l[rt] = s;
          } else {
#pragma unroll
            for (int r = 0; r < 16; ++r)
              c += step0 + l32 <= limit_of(row0 + rt * 32 + element(r)) ? fast_exp2(__builtin_fmaf(acc[r], kLogitScale, nlse[rt][r])) : 0.f;
          }
        }
        if constexpr (PASS == 2) {
          c = halves_sum(c, c);
          if (half == 0) s_sum[t % kSumTiles][rgi][step * 32 + l32] = c;
        }
      }
      if constexpr (PASS == 2) {
        __syncthreads();
        flush(t, t + 1);
      }
    }

    tile_barrier<0>();                    // no copy is in flight and nobody reads a tile any more
    if constexpr (PASS == 1) {
      // the two lanes that share a row, then the wavefronts that share the row group
      float* s_ml = reinterpret_cast<float*>(s_keys[0]);    // [ks][rgi][32 NRT rows][2]
#pragma unroll
      for (int rt = 0; rt < NRT; ++rt) {
        const float mm = fmaxf(m[rt], __shfl_xor(m[rt], 32));
        const float own = l[rt] * fast_exp2(m[rt] - mm), ll = halves_sum(own, own);
        if (half == 0) {
          float* p = s_ml + ((ks * RGW + rgi) * 32 * NRT + rt * 32 + l32) * 2;
          p[0] = mm;
          p[1] = ll;
        }
      }
      __syncthreads();
      if (tid < kRows) {
        const int row = sweep * kRows + tid;
        if (row < a.R) {
          float mm = kNegBig, ll = 0.f;
#pragma unroll
          for (int k = 0; k < kSplit; ++k) mm = fmaxf(mm, s_ml[(k * kRows + tid) * 2]);
#pragma unroll
          for (int k = 0; k < kSplit; ++k) ll += s_ml[(k * kRows + tid) * 2 + 1] * fast_exp2(s_ml[(k * kRows + tid) * 2] - mm);
          *reinterpret_cast<float2*>(a.row_part + (blk * a.row_slots + row) * 2) = make_float2(mm, ll);
        }
      }
    }
    __syncthreads();                      // before the next sweep's keys overwrite the buffers
  }

  if constexpr (kSquares) {
    // threads with the same piece of the key: prow differs; thread (prow, piece) holds channels 8 piece .. + 7
    float* s_k = reinterpret_cast<float*>(s_keys[0]);       // [16 prow][128]
#pragma unroll
    for (int j = 0; j < 8; ++j) s_k[prow * kHeadDim + piece * 8 + j] = ksq[j];
    __syncthreads();
    if (tid < kHeadDim) {
      float s = 0.f;
#pragma unroll
      for (int k = 0; k < 16; ++k) s += s_k[k * kHeadDim + tid];
      a.ksq_part[blk * kHeadDim + tid] = s;
    }
    __syncthreads();
  }
  }   // items of the run
}

// log-sum-exp of every window row over the runs of its item (log2 domain): 16 rows per workgroup, 16 threads stride
// over a row's runs; the workgroups behind them: the channel weights, where they are wanted
__global__ __launch_bounds__(256) void row_lse_kernel(WeightArgs a, float* __restrict__ w_ch) {
  if (static_cast<int>(blockIdx.x) * 16 >= a.row_slots) {
    channel_weights(a, w_ch, blockIdx.y, static_cast<int>(blockIdx.x) - a.row_slots / 16);
    return;
  }
  __shared__ float s_m[16][17], s_l[16][17];
  const int item = blockIdx.y;
  const int lr = threadIdx.x & 15, sub = threadIdx.x >> 4;
  const int r = blockIdx.x * 16 + lr;
  int slot0;
  const int n = item_slots(a, item, &slot0);
  const float2* p = reinterpret_cast<const float2*>(a.row_part) + static_cast<int64_t>(slot0) * a.row_slots + r;
  float m = kNegBig, l = 0.f;
  if (r < a.R) {
    for (int b0 = sub; b0 < n; b0 += 16 * 8) {     // eight independent loads in flight
      float2 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        v[u] = make_float2(kNegBig, 0.f);
        if (b0 + 16 * u < n) v[u] = p[static_cast<int64_t>(b0 + 16 * u) * a.row_slots];
      }
      float mb = m;
#pragma unroll
      for (int u = 0; u < 8; ++u) mb = fmaxf(mb, v[u].x);
      l *= fast_exp2(m - mb);
#pragma unroll
      for (int u = 0; u < 8; ++u) l += v[u].y * fast_exp2(v[u].x - mb);
      m = mb;
    }
  }
  s_m[sub][lr] = m;
  s_l[sub][lr] = l;
  __syncthreads();
  if (sub == 0) {
    float mm = kNegBig;
#pragma unroll
    for (int k = 0; k < 16; ++k) mm = fmaxf(mm, s_m[k][lr]);
    float ll = 0.f;
#pragma unroll
    for (int k = 0; k < 16; ++k) ll += s_l[k][lr] * fast_exp2(s_m[k][lr] - mm);
    // a padded row has no visible key: give it +inf so that exp2(x - lse) = 0
    a.lse[static_cast<int64_t>(item) * a.row_slots + r] = (ll > 0.f) ? mm + __log2f(ll) : INFINITY;
  }
}

// AvgPool1d(kernel, stride 1, zero padding kernel/2, divisor kernel) along the keys of each item
// (kernel odd, at most 15).  256 PER keys per workgroup; every load is issued before anything waits, and each key is read
// once: with a thread per key and its neighbours read from memory 2.9M keys took 13.7 us.
template <int PER>
__global__ __launch_bounds__(256) void pool_kernel(const float* __restrict__ w_raw, float* __restrict__ w_out,
                                                   int kernel, Batch batch) {
  constexpr int kRows = 256 * PER, kMostRadius = 7;
  __shared__ float s_w[kRows + 2 * kMostRadius];
  const ItemOf it(batch, blockIdx.y);
  const int T = it.T;
  const int t0 = blockIdx.x * kRows, tid = threadIdx.x;
  if (t0 >= T) return;
  const float* w = w_raw + it.off;
  float* out = w_out + it.off;
  const int r = kernel / 2, first = t0 - r;
  float v[PER + 1];
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int u = first + 256 * j + tid;
    v[j] = u >= 0 && u < T ? w[u] : 0.f;
  }
  const int last = first + kRows + tid;
  v[PER] = tid < 2 * r && last < T ? w[last] : 0.f;
#pragma unroll
  for (int j = 0; j < PER; ++j) s_w[256 * j + tid] = v[j];
  if (tid < 2 * r) s_w[kRows + tid] = v[PER];
  __syncthreads();
  float s[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) s[j] = 0.f;
  for (int k = 0; k <= 2 * r; ++k)
#pragma unroll
    for (int j = 0; j < PER; ++j) s[j] += s_w[256 * j + tid + k];
  const float count = static_cast<float>(kernel);
#pragma unroll
  for (int j = 0; j < PER; ++j)
    if (t0 + 256 * j + tid < T) out[t0 + 256 * j + tid] = s[j] / count;
}

// R in whole sweeps of row groups
int row_slots_of(int R) { return R <= 64 ? 64 : R <= 128 ? 128 : (R + 255) / 256 * 256; }

template <int NRT, int RGW>
void launch_passes(const WeightArgs& a, float* w_ch, hipStream_t st) {
  if (w_ch) hipLaunchKernelGGL((weights_kernel<1, NRT, RGW, true>), dim3(a.workgroups), dim3(256), 0, st, a);
  else hipLaunchKernelGGL((weights_kernel<1, NRT, RGW, false>), dim3(a.workgroups), dim3(256), 0, st, a);
  if (a.lse) hipLaunchKernelGGL(row_lse_kernel, dim3(a.row_slots / 16 + (w_ch ? kHeadDim / kChannelPart : 0), a.n_items), dim3(256), 0, st, a, w_ch);
  if (!a.w_ch) hipLaunchKernelGGL((weights_kernel<2, NRT, RGW, false>), dim3(a.sum_workgroups), dim3(256), 0, st, a);
}
// (A function of its own, used behind the others, so that its kernels stand behind theirs in the code: between them they made 8 x 128K
// tokens 1.5 % slower, by where the other kernels, the same to the instruction, came to lie: 233.5 -> 238 us a pass.)
template <int NRT, int RGW>
void launch_pass2_with_channels(const WeightArgs& a, hipStream_t st) {
  hipLaunchKernelGGL((weights_kernel<2, NRT, RGW, true>), dim3(a.sum_workgroups + a.n_items * (kHeadDim / kChannelPart)), dim3(256), 0, st, a);
}

}  // namespace

// scratch layout (floats): row_part | lse | w_raw | ksq_part
size_t weights_scratch_floats(int64_t n_tiles, int64_t n_items, int64_t total_tokens, int R, bool want_ch) {
  const size_t slots = static_cast<size_t>(workgroups_of(n_tiles, kPass1PerCu)) + n_items;
  return slots * row_slots_of(R) * 2 + static_cast<size_t>(n_items) * row_slots_of(R) + static_cast<size_t>(total_tokens) +
         (want_ch ? slots * kHeadDim : 0) + 64;
}

// raw: where the weights before the pooling are (scratch), for a caller that pools them; w_tok is left alone then.
hipError_t launch_weights(const rdkv_config& cfg, const Batch& batch, int64_t n_tiles, int64_t n_items, int64_t total_tokens,
                          int max_T, const uint16_t* K, const uint16_t* Q_obs, float* w_tok, float* w_ch,
                          float* scratch, const float** raw, hipStream_t st) {
  if (n_items == 0 || max_T == 0) return hipSuccess;
  WeightArgs a;
  a.K = K; a.Q = Q_obs; a.batch = batch;
  a.hq = cfg.hq; a.hkv = cfg.hkv; a.g = cfg.hq / cfg.hkv; a.s_obs = cfg.s_obs;
  a.R = a.g * cfg.s_obs; a.row_slots = row_slots_of(a.R); a.causal = cfg.causal ? 1 : 0;
  a.n_items = static_cast<int32_t>(n_items); a.n_tiles = static_cast<int32_t>(n_tiles);
  const RunPlan runs = run_plan(n_tiles, (max_T + kKeyTile - 1) / kKeyTile, a.R, kPass1PerCu);
  a.workgroups = runs.workgroups;
  const int64_t slots = a.workgroups + n_items;
  a.row_part = scratch;
  a.lse = a.row_part + slots * a.row_slots * 2;
  a.w_raw = a.lse + n_items * a.row_slots;
  // An item of few runs needs no launch of its own for the log-sum-exp: pass 2 makes it while its first keys arrive.  Launch +
  // pass 2 against pass 2: 16 x 1K tokens 3.9 + 16.0 -> 16.0 us, 4 x 8K (17 runs) 4.2 + 20.1 -> 21.5, 128 items of 20K tokens
  // 5.4 + 185.6 -> 188.8.  Eight items have 65 runs each, and every workgroup would read them: 32K tokens 4.7 + 18.5 -> 22.7, 128K
  // tokens and 256 rows 5.3 + 78 -> 88.  The channel weights go along with whichever launch makes it: with
  // pass 2 passes over 5 x 1K tokens of 4 heads 126.7 -> 122.2 us, 11 x 0.8K of 8 128.5 -> 126.4, 5 x 8K of 4 111.2 -> 110.2.
  if (lse_in_second_pass(runs, n_items, a.R, w_ch != nullptr)) a.lse = nullptr;
  a.sum_workgroups = workgroups_of(n_tiles, kPass2PerCu);
  a.w_ch = a.lse ? nullptr : w_ch;
  a.ksq_part = w_ch ? a.w_raw + total_tokens : nullptr;
  if (a.R <= 64) launch_passes<1, 2>(a, w_ch, st);
  else if (a.R <= 128) launch_passes<2, 2>(a, w_ch, st);
  else launch_passes<2, 4>(a, w_ch, st);
  if (a.w_ch) {
    if (a.R <= 64) launch_pass2_with_channels<1, 2>(a, st);
    else if (a.R <= 128) launch_pass2_with_channels<2, 2>(a, st);
    else launch_pass2_with_channels<2, 4>(a, st);
  }
  if (raw) {
    *raw = a.w_raw;
  } else if (cfg.pool_kernel > 1) {
    // enough workgroups for the chip first, then several keys per thread
    const bool wide = n_items * ((max_T + 1023) / 1024) >= 1024;
    const unsigned per_wg = wide ? 1024 : 256;
    const dim3 grid((static_cast<unsigned>(max_T) + per_wg - 1) / per_wg, static_cast<unsigned>(n_items));
    if (wide) hipLaunchKernelGGL(pool_kernel<4>, grid, dim3(256), 0, st, a.w_raw, w_tok, cfg.pool_kernel, batch);
    else hipLaunchKernelGGL(pool_kernel<1>, grid, dim3(256), 0, st, a.w_raw, w_tok, cfg.pool_kernel, batch);
  } else {
    hipError_t e = hipMemcpyAsync(w_tok, a.w_raw, total_tokens * sizeof(float), hipMemcpyDeviceToDevice, st);
    if (e != hipSuccess) return e;
  }
  return hipGetLastError();
}

}  // namespace rdkv
