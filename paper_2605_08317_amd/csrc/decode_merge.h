// Log-sum-exp merge of the split partials of a decode step (the last step of Eq. 7's evaluation as a split-K
// flash-decode) inside the decode launch itself: one launch per step instead of a split launch and a merge launch.
//
// Memory across the chip's eight L2 caches: partials are written and read with agent-scope accesses, which go through to
// memory instead of staying in one XCD's L2.  Either way of merging has a fixed summation order (slot order), so results do
// not depend on which chunk happens to end last.
//
// Large launches count (arrive_and_merge): every workgroup stores its chunk's partial, waits until the stores have drained,
// announces it on the item's arrival counter, and the workgroup that completes an item merges its partials and resets the
// counter.
//
// Small launches with up to 128 query heads look (merge_part; merge_parts in rdkv_api.hip says where the line lies): behind the
// chunks they have workgroups that only merge, each some of an item's output channels.  A word of a partial is its own arrival
// flag: between steps every word of the workspace holds kAbsent, a NaN that a partial never holds (`present`), and the merging
// wavefront puts it back once it has read a word.  What that saves is two memory round trips between a chunk's last store and
// the merge (drain, counter; 20 arrivals at once queue for 1.4 us) and a merge in one workgroup per item with eight slots per
// thread: from the last partial's store to the end of the launch 4.3 us counted, 1.7 so (time stamps, 164 chunks).
// Launches of 30, 164 and 178 chunks with 2 to 8 items 7.0 -> 5.1, 9.5 -> 6.7 and 10.7 -> 9.2 us, 208 channel-wise ones
// 15.2 -> 12.3 (replayed from a graph).
// In larger launches the merging workgroups come too late, one behind the other in what slots the chunks leave (16 ragged
// sequences with 8 query heads 43.7 us counted, 46.8 looked at; 16 channel-wise ones 77.6, 77.8).
//
// What bounds the wait of a merging workgroup.  Workgroups are dispatched in the order of the grid on each XCD, but an item's
// chunks are on all of them, and launches on other streams and of other processes share them: merging workgroups of several
// launches could hold all places of the XCDs that each other's chunks need.  So a merging wavefront waits for chunks that may
// have no place yet for a while only (MergeArgs::looks), then hands its block over (give_up), and holds no place any more.
//   Each line has a state word, of which either side clears a bit of its own in one atomic that returns what the other has
// cleared: a chunk's wavefront when it is through with its tiles (that is also the news that it ends soon; the answer is there
// by the time that its partial is stored), a merging wavefront when it gives up.  Where the chunk came first, its workgroup runs
// and waits for nothing, and a merging wavefront may wait for its partial: it does so once all chunks of the item have come, and,
// after it has given up, for those that had.  Then it sets the block's hand-over word and looks once more.  Where the merging
// wavefront came first, the chunk's wavefront finds it out, waits until its own stores have landed, reads the hand-over word, and
// if it is set looks once.  Of all these take the one whose partial landed last: if it read the word before it was set, all
// partials had landed by then, and the merging wavefront's last look finds them; otherwise its own look does.  Who finds all of
// them takes the block by a compare-and-exchange on the hand-over word, and only the taker puts words back and writes the
// output.  No words are put back before every chunk's bit is cleared, so no atomic is under way then.
#pragma once
#include "rdkv_internal.h"
#include "wave_ops.h"

namespace rdkv {

struct MergeArgs {
  float* part_acc;     // [slots][g][128] unnormalised partial outputs; launches that look: [slots][g] look records
  float* part_ml;      // [slots][g][2]   running maximum (log2 domain) and sum of each partial (launches that count)
  int32_t* arrive;     // [items] arrival counters, zero between steps (launches that count)
  float* out;          // [batch][hq][128]
  float* lse;          // [batch][hq] or null
  int32_t g;           // query heads per KV head: item i (sequence x KV head) owns output rows i g .. i g + g - 1
  int32_t parts;       // merging workgroups of an item, 8 g / parts blocks each, a wavefront each; 0: the launch counts
  int32_t looks;       // how often they look before they leave their blocks to the chunks (rdkv_cache::looks)
};

inline hipError_t launch_decode_mixed(const Chunk* chunks, int n_chunks, const uint8_t* arena, const ItemK* items_k,
                                      int max_words, int max_steps, int max_qsteps, const uint16_t* q,
                                      const MergeArgs& ma, const int32_t* tail_len, int per_unit, int waves,
                                      hipStream_t st) {
  const bool hs2 = ma.g > 4, lng = max_words > 32;
  return (hs2 ? (lng ? launch_decode_mixed_hs2_long1 : launch_decode_mixed_hs2_long0)
              : (lng ? launch_decode_mixed_hs1_long1 : launch_decode_mixed_hs1_long0))(
      chunks, n_chunks, arena, items_k, max_words, max_steps, max_qsteps, q, ma, tail_len, per_unit, waves, st);
}

namespace merge {

constexpr float kNegBig = -1.0e30f;

constexpr uint32_t kAbsent = 0xFFFFFFFFu;
// A line's state word: bits that are cleared once a step.  An item's hand-over word for a block (state word of a second kind, in
// the line of its first slot): kAbsent, or kReady from when the block is left to the chunks until some wavefront takes it.
constexpr uint32_t kEndsSoon = 1, kGivenUp = 2;
constexpr uint32_t kReady = 0;
constexpr int kStateWord = 18, kHandOverWord = 19;
constexpr int kMostLooks = 1 << 20;       // at chunks that run (seconds): should two steps share a workspace, which is not allowed
constexpr int kSc1 = 16;                  // cache policy of the buffer accesses: agent scope

using uint4v = __attribute__((ext_vector_type(4))) unsigned;
using uint2v = __attribute__((ext_vector_type(2))) unsigned;

// v, with another NaN in place of kAbsent
__device__ __forceinline__ float present(float v) {
  return __float_as_uint(v) == kAbsent ? __uint_as_float(0x7FC00000u) : v;
}
__device__ __forceinline__ void store_agent(float* p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_agent2(float* p, float v0, float v1) {     // (p: a multiple of eight bytes)
  __hip_atomic_store(reinterpret_cast<uint64_t*>(p),
                     static_cast<uint64_t>(__float_as_uint(v0)) | (static_cast<uint64_t>(__float_as_uint(v1)) << 32),
                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A look record: the partial of a slot and head in kBlocks blocks of 16 channels, which have a reading wavefront each.  A block
// is a line of 128 bytes: [16] accumulators, running maximum, sum, state, hand-over (in the line of the item's first slot);
// so that a reader's loads of a block are one request.
constexpr int kBlocks = 8, kBlockFloats = 32, kRecordFloats = kBlocks * kBlockFloats;
__device__ __forceinline__ float* look_record(const MergeArgs& ma, int slot, int head, int block) {
  return ma.part_acc + (static_cast<int64_t>(slot) * ma.g + head) * kRecordFloats + block * kBlockFloats;
}

// (block: counted over the heads of the item)
__device__ __forceinline__ uint32_t* look_word(const MergeArgs& ma, int slot, int block, int word) {
  return reinterpret_cast<uint32_t*>(look_record(ma, slot, block / kBlocks, block % kBlocks) + word);
}
__device__ __forceinline__ uint32_t clear_state(const MergeArgs& ma, int slot, int block, uint32_t bit) {
  return __hip_atomic_fetch_and(look_word(ma, slot, block, kStateWord), ~bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool take_block(const MergeArgs& ma, int slot0, int block) {
  uint32_t ready = kReady;
  bool mine = false;
  if ((threadIdx.x & 63) == 0)
    mine = __hip_atomic_compare_exchange_strong(look_word(ma, slot0, block, kHandOverWord), &ready, kAbsent, __ATOMIC_RELAXED,
                                                __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return __any(mine);
}

// Every thread calls this after its last store_agent of the partial and before the workgroup barrier that precedes
// arrive_and_merge(): agent-scope stores are written through to memory, so once the wave's store counter has drained
// they are visible to every XCD.  (A release fence would add a write-back of the whole L2, which has nothing of
// ours to write back and costs the launch tens of microseconds when hundreds of workgroups issue it.)
__device__ __forceinline__ void partial_stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// The merge proper for G query heads per KV head: thread = (slot group, four neighbouring channels of a head).  Every load
// of a thread's slots is issued before anything waits (one memory round trip for up to SG * kBatch slots); each slot group
// reduces its slots with running maxima, and the SG groups are combined through LDS.  Sixteen bytes of a partial and one
// (maximum, sum) pair per load -- with one channel and all heads per thread (96 loads instead of 16 at g = 4) the merge of
// 21 slots took 2.75 us of a 12.3 us launch.
// THROUGH: the output goes through to memory like the partials (rows that other XCDs have stored to in this launch)
template <int NT, int G, int kBatch = 8, bool THROUGH = false>
__device__ __forceinline__ void merge_item(const MergeArgs& ma, int item, int slot0, int nslots, float* smem) {
  constexpr int kCols = G * kHeadDim / 4;
  constexpr int SG = NT / kCols;
  static_assert(SG >= 1, "a workgroup covers a slot's partial");
  const int tid = threadIdx.x;
  const int col = tid & (kCols - 1), sg = tid / kCols, hd = col >> 5;
  float* s_m = smem + 16;                   // [SG][G]
  float* s_l = s_m + SG * G;                // [SG][G]
  float* s_red = smem + 16 + 2 * SG * G;    // [SG][G][128]
  // loads past the last slot return zeros (the buffer's bounds)
  const auto acc_rsrc = __builtin_amdgcn_make_buffer_rsrc(ma.part_acc + static_cast<int64_t>(slot0) * G * kHeadDim, 0,
                                                          nslots * G * kHeadDim * 4, 0x00027000);
  const auto ml_rsrc = __builtin_amdgcn_make_buffer_rsrc(ma.part_ml + static_cast<int64_t>(slot0) * G * 2, 0,
                                                         nslots * G * 8, 0x00027000);
  float m_run = kNegBig, l_run = 0.f, o_run[4] = {0.f, 0.f, 0.f, 0.f};
  for (int s0 = sg; s0 < nslots; s0 += SG * kBatch) {
    uint4v a[kBatch];
    uint2v ml[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int s = s0 + u * SG;
      ml[u] = __builtin_amdgcn_raw_buffer_load_b64(ml_rsrc, (s * G + hd) * 8, 0, kSc1);
      a[u] = __builtin_amdgcn_raw_buffer_load_b128(acc_rsrc, (s * kCols + col) * 16, 0, kSc1);
    }
    float mb = m_run, mv[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      mv[u] = s0 + u * SG < nslots ? __uint_as_float(ml[u].x) : kNegBig;
      mb = fmaxf(mb, mv[u]);
    }
    const float f0 = __builtin_amdgcn_exp2f(m_run - mb);
    l_run *= f0;
#pragma unroll
    for (int k = 0; k < 4; ++k) o_run[k] *= f0;
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const float f = __builtin_amdgcn_exp2f(mv[u] - mb);
      l_run = __builtin_fmaf(__uint_as_float(ml[u].y), f, l_run);
#pragma unroll
      for (int k = 0; k < 4; ++k) o_run[k] = __builtin_fmaf(__uint_as_float(a[u][k]), f, o_run[k]);
    }
    m_run = mb;
  }
  const int64_t qh0 = static_cast<int64_t>(item) * G;
  if constexpr (SG == 1) {
    float* o = ma.out + qh0 * kHeadDim + 4 * col;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float v = l_run > 0.f ? o_run[k] / l_run : 0.f;
      if constexpr (THROUGH) store_agent(o + k, v); else o[k] = v;
    }
    if ((col & 31) == 0 && ma.lse != nullptr)
      ma.lse[qh0 + hd] = l_run > 0.f ? (m_run + __log2f(l_run)) * 0.6931471805599453f : -INFINITY;
    return;
  }
  *reinterpret_cast<float4*>(s_red + (sg * kCols + col) * 4) = make_float4(o_run[0], o_run[1], o_run[2], o_run[3]);
  if ((col & 31) == 0) { s_m[sg * G + hd] = m_run; s_l[sg * G + hd] = l_run; }
  __syncthreads();
  for (int idx = tid; idx < G * kHeadDim; idx += NT) {
    const int h = idx >> 7;
    float mm = kNegBig;
#pragma unroll
    for (int k = 0; k < SG; ++k) mm = fmaxf(mm, s_m[k * G + h]);
    float l = 0.f, t = 0.f;
#pragma unroll
    for (int k = 0; k < SG; ++k) {
      const float f = __builtin_amdgcn_exp2f(s_m[k * G + h] - mm);
      l = __builtin_fmaf(s_l[k * G + h], f, l);
      t = __builtin_fmaf(s_red[k * G * kHeadDim + idx], f, t);
    }
    const float v = l > 0.f ? t / l : 0.f;
    if constexpr (THROUGH) store_agent(ma.out + qh0 * kHeadDim + idx, v); else ma.out[qh0 * kHeadDim + idx] = v;
    if ((idx & 127) == 0 && ma.lse != nullptr)
      ma.lse[qh0 + h] = l > 0.f ? (mm + __log2f(l)) * 0.6931471805599453f : -INFINITY;
  }
}

// Called by all NT threads of a workgroup after a barrier that follows partial_stores_done().  Returns after the
// item's output rows are written if this workgroup arrived last, at once otherwise.
// smem: merge_lds_floats(NT) floats of 16-byte aligned LDS that nothing else uses any more.
// GMAX: the most query heads per KV head the calling kernel is built for (larger merges are not compiled into it)
template <int NT, int GMAX = 8>
__device__ __forceinline__ void arrive_and_merge(const MergeArgs& ma, int item, int slot0, int nslots, int g,
                                                 float* smem) {
  static_assert(NT % 128 == 0 && NT >= 128, "the merge assigns 128 channel threads per slot group");
  const int tid = threadIdx.x;
  int* s_flag = reinterpret_cast<int*>(smem);
  if (tid == 0) {
    const int old = __hip_atomic_fetch_add(ma.arrive + item, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *s_flag = old == nslots - 1;
  }
  __syncthreads();
  if (*s_flag == 0) return;
  // the partials are read with agent-scope loads, which do not hit stale lines of this XCD's caches
  if constexpr (GMAX > 4) {
    if (g > 4) merge_item<NT, 8>(ma, item, slot0, nslots, smem);
  }
  switch (g) {
    case 1: merge_item<NT, 1>(ma, item, slot0, nslots, smem); break;
    case 2: merge_item<NT, 2>(ma, item, slot0, nslots, smem); break;
    case 4: merge_item<NT, 4>(ma, item, slot0, nslots, smem); break;
    default: break;
  }
  if (tid == 0) __hip_atomic_store(ma.arrive + item, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// All chunks of an item say that they end soon, in the lines of a block.  ONCE: at the first look; otherwise after at most looks
// of them.
template <bool ONCE>
__device__ __forceinline__ bool all_end_soon(const MergeArgs& ma, int slot0, int nslots, int block) {
  constexpr int kLoads = 4;
  const int step = ma.g * kRecordFloats * 4;      // bytes from slot to slot
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(ma.part_acc + static_cast<int64_t>(slot0) * ma.g * kRecordFloats, 0,
                                                      nslots * step, 0x00027000);
  const int at = (threadIdx.x & 63) * step + (block * kBlockFloats + kStateWord) * 4;
  int tries = 0;
  for (int base = 0; base < nslots; base += 64 * kLoads)
    for (;;) {
      uint32_t state[kLoads], most = 0;
#pragma unroll
      for (int u = 0; u < kLoads; ++u)            // (past the last slot: zero)
        state[u] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, (base + u * 64) * step + at, 0, kSc1);
      asm volatile("" ::: "memory");              // (load again next time)
#pragma unroll
      for (int u = 0; u < kLoads; ++u) most = max(most, state[u] | ~kEndsSoon);
      if (!__any(most == kAbsent)) break;
      if (ONCE || ++tries >= ma.looks) return false;
    }
  return true;
}

// One wavefront, after all_end_soon: a block of 16 channels, counted over the heads of the item.
// lane = (slot group of sixteen, four neighbouring channels); BATCH slots of a lane at a time, all loads of a batch in flight
// together and repeated until none of their words is absent; then the slot groups are added across the lanes.  No LDS and no
// barrier: what a workgroup's wavefronts exchange they would wait for (a slot group per half wavefront and the rest through
// LDS took 1.2 us from the last word's arrival, this 0.5).  What bounds it then are requests: two per slot and block, eight
// wavefronts of 32 workgroups, made 16 MB layers 10.8 us; a line per block and 64 workgroups 9.3, 128 of them 9.2.
// ONCE: one look at a block that its merging wavefront left to the chunks; nothing happens if words are still absent, or if
// another wavefront has taken the block.
template <int BATCH, bool ONCE>
__device__ __forceinline__ void merge_block(const MergeArgs& ma, int item, int slot0, int nslots, int block) {
  constexpr int SG = 16;
  const int lane = threadIdx.x & 63, sg = lane >> 2, col = lane & 3;
  const int step = ma.g * kRecordFloats * 4;      // bytes from slot to slot
  // loads past the last slot return zeros, stores there are dropped (the buffer's bounds)
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(ma.part_acc + static_cast<int64_t>(slot0) * ma.g * kRecordFloats, 0,
                                                      nslots * step, 0x00027000);
  const int ml_at = block * (kBlockFloats * 4) + 64, acc_at = block * (kBlockFloats * 4) + col * 16;
  const auto put_back = [&](int base) __attribute__((always_inline)) {
    const uint4v absent = {kAbsent, kAbsent, kAbsent, kAbsent};
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
      const int s = (base + u * SG + sg) * step;
      __builtin_amdgcn_raw_buffer_store_b128(absent, rsrc, s + acc_at, 0, kSc1);
      if (col == 0) __builtin_amdgcn_raw_buffer_store_b128(absent, rsrc, s + ml_at, 0, kSc1);
    }
  };
  struct Slots {
    uint4v a[BATCH];
    uint2v ml[BATCH];
  };
  Slots x, y;                                     // two looks under way, half a round trip apart
  float m_run = kNegBig, l_run = 0.f, o_run[4] = {0.f, 0.f, 0.f, 0.f};
  int tries = 0;
  for (int base = 0; base < nslots; base += SG * BATCH) {
    const auto load = [&](Slots& v) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < BATCH; ++u) {
        const int s = (base + u * SG + sg) * step;
        v.ml[u] = __builtin_amdgcn_raw_buffer_load_b64(rsrc, s + ml_at, 0, kSc1);
        v.a[u] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, s + acc_at, 0, kSc1);
      }
      asm volatile("" ::: "memory");
    };
    const auto complete = [&](const Slots& v) __attribute__((always_inline)) {
      uint32_t most = 0;                          // kAbsent is the largest word
#pragma unroll
      for (int u = 0; u < BATCH; ++u) {
        most = max(max(most, v.ml[u].x), v.ml[u].y);
        most = max(max(most, v.a[u].x), v.a[u].y);
        most = max(max(most, v.a[u].z), v.a[u].w);
      }
      return !__any(most == kAbsent);
    };
    Slots z;
    load(x);
    if constexpr (ONCE) {
      if (!complete(x)) return;
      z = x;
    } else {
      for (;;) {
        load(y);
        if (complete(x) || ++tries >= kMostLooks) { z = x; break; }
        load(x);
        if (complete(y) || ++tries >= kMostLooks) { z = y; break; }
      }
      put_back(base);
    }
    float mb = m_run, mv[BATCH];
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
      mv[u] = base + u * SG + sg < nslots ? __uint_as_float(z.ml[u].x) : kNegBig;
      mb = fmaxf(mb, mv[u]);
    }
    const float f0 = __builtin_amdgcn_exp2f(m_run - mb);
    l_run *= f0;
#pragma unroll
    for (int k = 0; k < 4; ++k) o_run[k] *= f0;
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
      const float f = __builtin_amdgcn_exp2f(mv[u] - mb);
      l_run = __builtin_fmaf(__uint_as_float(z.ml[u].y), f, l_run);
#pragma unroll
      for (int k = 0; k < 4; ++k) o_run[k] = __builtin_fmaf(__uint_as_float(z.a[u][k]), f, o_run[k]);
    }
    m_run = mb;
  }
  if constexpr (ONCE) {
    if (!take_block(ma, slot0, block)) return;
    for (int base = 0; base < nslots; base += SG * BATCH) put_back(base);
  }
  const float mm = head_max(m_run);
  const float f = __builtin_amdgcn_exp2f(m_run - mm);
  const float l = head_sum(l_run * f);
  // the sums over the slot groups, the four channels turned into the four rows of lanes on the way
  float o[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) o[k] = o_run[k] * f;
  swap_rows(o[0], o[1]);
  swap_rows(o[2], o[3]);
  float lo = o[0] + o[1], hi = o[2] + o[3];
  swap_halves(lo, hi);
  float v = lo + hi;
  v += dpp_f32<0x124>(v);
  v += dpp_f32<0x128>(v);
  if ((lane & 12) == 0)
    ma.out[static_cast<int64_t>(item) * ma.g * kHeadDim + block * 16 + 4 * col + (lane >> 4)] = l > 0.f ? v / l : 0.f;
  if (lane == 0 && block % kBlocks == 0 && ma.lse != nullptr)
    ma.lse[static_cast<int64_t>(item) * ma.g + block / kBlocks] = l > 0.f ? (mm + __log2f(l)) * 0.6931471805599453f : -INFINITY;
  // The look that was not needed is still on its way: its registers must not be used for anything before (that would wait for
  // it: 0.8 us).
  if constexpr (!ONCE) {
#pragma unroll
    for (int u = 0; u < BATCH; ++u) asm volatile("" ::"v"(x.a[u]), "v"(x.ml[u]), "v"(y.a[u]), "v"(y.ml[u]));
  }
}

// slots of a lane at a time: the same whoever merges, since the order of the sums depends on it
template <bool ONCE>
__device__ __forceinline__ void merge_block(const MergeArgs& ma, int item, int slot0, int nslots, int block) {
  if (nslots <= 32) merge_block<2, ONCE>(ma, item, slot0, nslots, block);
  else merge_block<4, ONCE>(ma, item, slot0, nslots, block);
}
// (a look at the state words as well: no atomic of a chunk may be under way when words are put back)
__device__ __forceinline__ void merge_if_complete(const MergeArgs& ma, int item, int slot0, int nslots, int block) {
  if (all_end_soon<true>(ma, slot0, nslots, block)) merge_block<true>(ma, item, slot0, nslots, block);
}

// lane -> a block of the heads whose partials this wavefront stores (heads wave, wave + NWV, ..; from 8 g on: none)
template <int NWV>
__device__ __forceinline__ int own_block() {
  const int lane = threadIdx.x & 63;
  return (static_cast<int>(threadIdx.x >> 6) + lane / kBlocks * NWV) * kBlocks + lane % kBlocks;
}

// A merging wavefront leaves its block to the chunks, except for what it need not be afraid of waiting for: the slots whose
// workgroups are through with their tiles.
__device__ __forceinline__ void give_up(const MergeArgs& ma, int slot0, int nslots, int block) {
  const int lane = threadIdx.x & 63;
  for (int s = lane; s < nslots; s += 64) {
    if (clear_state(ma, slot0 + s, block, kGivenUp) & kEndsSoon) continue;
    for (int tries = 0; tries < kMostLooks; ++tries) {
      uint32_t most = 0;
      for (int w = 0; w < kStateWord; ++w)
        most = max(most, __hip_atomic_load(look_word(ma, slot0 + s, block, w), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
      if (most != kAbsent) break;
    }
  }
  if (lane == 0)
    __hip_atomic_store(look_word(ma, slot0, block, kHandOverWord), kReady, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  partial_stores_done();
}

// A merging workgroup of NWV wavefronts (a chunk of tier kTierMerge): part ch.row0 of the item's blocks, one a wavefront.
template <int NWV>
__device__ __forceinline__ void merge_part(const MergeArgs& ma, const Chunk& ch) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int blocks = ma.g * kBlocks / ma.parts, block = ch.row0 * blocks + wave;
  if (wave >= blocks) return;
  // "Ends soon" first: the loads of whole partials would take their bandwidth from the chunks.  (It takes a chunk 1 us from
  // there to its stores, and the news a little less to come here.)
  if (all_end_soon<false>(ma, ch.slot0, ch.nslots, block)) {
    merge_block<false>(ma, ch.item, ch.slot0, ch.nslots, block);
  } else {
    give_up(ma, ch.slot0, ch.nslots, block);
    merge_if_complete(ma, ch.item, ch.slot0, ch.nslots, block);
  }
}

// The end of a chunk's wavefront in a launch that looks, after store_partial.  state: of its heads' blocks, which it cleared a
// bit of when it was through with its tiles (ends_soon).  One look at each block that its merging wavefront had left by then.
template <int NWV>
__device__ __forceinline__ void merge_left(const MergeArgs& ma, int item, int slot0, int nslots, uint32_t state) {
  if (__builtin_expect(!__any((state & kGivenUp) == 0), true)) return;
  partial_stores_done();
  const int block = own_block<NWV>();
  uint32_t word = kAbsent;
  if ((state & kGivenUp) == 0)
    word = __hip_atomic_load(look_word(ma, slot0, block, kHandOverWord), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  for (uint64_t lanes = __ballot(word == kReady); lanes != 0; lanes &= lanes - 1)
    merge_if_complete(ma, item, slot0, nslots, __builtin_amdgcn_readlane(block, __builtin_ctzll(lanes)));
}

// LDS floats arrive_and_merge needs for NT threads (a flag, at most NT / 32 maxima and sums, four sums per thread)
__host__ __device__ constexpr int merge_lds_floats(int nt) { return 16 + 2 * (nt / 32) + nt * 4; }

}  // namespace merge
}  // namespace rdkv
