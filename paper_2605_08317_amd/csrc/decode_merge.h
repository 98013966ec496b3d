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
// Small launches look (merge_part): behind the chunks they have workgroups that only merge, each some of an item's output
// channels.  A word of a partial is its own arrival flag: between steps every word of the workspace holds kAbsent, a NaN that a
// partial never holds (`present`), and the merging wavefront puts it back once it has read a word.  What that saves is two
// memory round trips between a chunk's last store and the merge (drain, counter; 20 arrivals at once queue for 1.4 us) and a
// merge in one workgroup per item with eight slots per thread: from the last partial's store to the end of the launch 4.3 us
// counted, 1.7 so (time stamps, 164 chunks).
// Launches of 30, 164 and 178 chunks with 2 to 8 items 7.0 -> 5.1, 9.5 -> 6.7 and 10.7 -> 9.2 us, 208 channel-wise ones
// 15.2 -> 12.3 (replayed from a graph).
// In large launches the merging workgroups come too late, one behind the other in what slots the chunks leave (16 ragged
// sequences with 8 query heads 43.7 us counted, 46.8 looked at; 16 channel-wise ones 77.6, 77.8).
//
// What bounds the wait of a merging workgroup.  Workgroups are dispatched in the order of the grid on each XCD, but an item's
// chunks are on all of them, and launches on other streams and of other processes share them: merging workgroups of several
// launches could hold all places of the XCDs that each other's chunks need.  So a merging wavefront waits for a chunk that has
// no place yet for a while only (MergeArgs::looks), then hands its blocks over (give_up), and holds no place any more.
//   Each line has a state word, of which either side clears a bit of its own in one atomic that returns what the other has
// cleared: a chunk's wavefront when it is through with its tiles (that is also the news that it ends soon; the answer is there
// by the time that its partial is stored, and costs the launch nothing), a merging wavefront when it gives up.  Where the chunk
// came first, its workgroup runs and waits for nothing, and the merging wavefront waits for its partial.  Then it sets
// the block's hand-over word and looks once more.  Where the merging wavefront came first, the chunk's wavefront finds it out,
// waits until its own stores have landed, reads the hand-over word, and if it is set looks once.  Of all these take the one
// whose partial landed last: if it read the word before it was set, all partials had landed by then, and the merging wavefront's
// last look finds them; otherwise its own look does.  Who finds all of them takes the block by a compare-and-exchange on the
// hand-over word, and only the taker puts words back and writes the output.  A partial is complete only with its chunk's bit
// cleared, so no atomic is under way when words are put back.
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
  int32_t parts;       // merging workgroups of an item, 8 g / parts blocks each
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
constexpr int kMostLooks = 1 << 20;       // of give_up at a running chunk, seconds: should two steps use one workspace at a time
constexpr int kSc1 = 16;                  // cache policy of the buffer accesses: agent scope

using uint4v = __attribute__((ext_vector_type(4))) unsigned;
using uint3v = __attribute__((ext_vector_type(3))) unsigned;
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
// kAbsent as long as the chunk has not said that it ends soon
__device__ __forceinline__ uint32_t ends_soon_or_absent(uint32_t state) { return state | ~kEndsSoon; }
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
template <int NT, int G>
__device__ __forceinline__ void merge_item(const MergeArgs& ma, int item, int slot0, int nslots, float* smem) {
  constexpr int kCols = G * kHeadDim / 4;
  constexpr int SG = NT / kCols;
  static_assert(SG >= 1, "a workgroup covers a slot's partial");
  constexpr int kBatch = 8;
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
    for (int k = 0; k < 4; ++k) o[k] = l_run > 0.f ? o_run[k] / l_run : 0.f;
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
    ma.out[qh0 * kHeadDim + idx] = l > 0.f ? t / l : 0.f;
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

// One wavefront: C blocks of 16 channels, block0 + k block_step counted over the heads of the item.
// lane = (slot group of sixteen, four neighbouring channels); BATCH slots of a lane at a time, all loads of a batch in flight
// together and repeated until none of their words is absent; then the slot groups are added across the lanes.  No LDS and no
// barrier: what a workgroup's wavefronts exchange they would wait for (a slot group per half wavefront and the rest through
// LDS took 1.2 us from the last word's arrival, this 0.5).  What bounds it then are requests: two per slot and block, eight
// wavefronts of 32 workgroups, made 16 MB layers 10.8 us; a line per block and 64 workgroups 9.3, 128 of them 9.2.
// False, and nothing is changed in memory: words are still absent after ma.looks looks, or (ONCE: one look at a block that a
// merging wavefront left) after that look, or another wavefront has taken the block.
template <int C, int BATCH, bool ONCE>
__device__ __forceinline__ bool merge_blocks(const MergeArgs& ma, int item, int slot0, int nslots, int block0, int block_step) {
  static_assert(!ONCE || C == 1, "blocks are taken one by one");
  constexpr int SG = 16;
  const int lane = threadIdx.x & 63, sg = lane >> 2, col = lane & 3;
  const int step = ma.g * kRecordFloats * 4;      // bytes from slot to slot
  // loads past the last slot return zeros, stores there are dropped (the buffer's bounds)
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(ma.part_acc + static_cast<int64_t>(slot0) * ma.g * kRecordFloats, 0,
                                                      nslots * step, 0x00027000);
  const auto ml_at = [&](int c) { return (block0 + c * block_step) * (kBlockFloats * 4) + 64; };
  const auto acc_at = [&](int c) { return (block0 + c * block_step) * (kBlockFloats * 4) + col * 16; };
  int tries = 0;
  // "Ends soon" first, until all slots of the first batch say so: the loads of whole partials would take their bandwidth from
  // the chunks.  (It takes a chunk 1 us from there to its stores, and the news a little less to come here.)
  if constexpr (!ONCE) {
    for (;;) {
      uint32_t soon[BATCH], most = 0;
#pragma unroll
      for (int u = 0; u < BATCH; ++u)             // (past the last slot: zero)
        soon[u] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, (u * SG + sg) * step + ml_at(0) + 8, 0, kSc1);
      asm volatile("" ::: "memory");              // (load again next time)
#pragma unroll
      for (int u = 0; u < BATCH; ++u) most = max(most, ends_soon_or_absent(soon[u]));
      if (!__any(most == kAbsent)) break;
      if (++tries >= ma.looks) return false;
    }
  }
  float m_run[C], l_run[C], o_run[C][4];
#pragma unroll
  for (int c = 0; c < C; ++c) {
    m_run[c] = kNegBig;
    l_run[c] = 0.f;
#pragma unroll
    for (int k = 0; k < 4; ++k) o_run[c][k] = 0.f;
  }
  struct Slots {
    uint4v a[C][BATCH];
    uint3v ml[C][BATCH];
  };
  // All words of the blocks absent again, once the last of them has been read: what gives up between two batches must leave
  // the first one to others.
  const auto put_back = [&]() __attribute__((always_inline)) {
    const uint4v absent = {kAbsent, kAbsent, kAbsent, kAbsent};
    for (int s = sg * step; s - sg * step < nslots * step; s += SG * step)
#pragma unroll
      for (int c = 0; c < C; ++c) {
        __builtin_amdgcn_raw_buffer_store_b128(absent, rsrc, s + acc_at(c), 0, kSc1);
        if (col == 0) __builtin_amdgcn_raw_buffer_store_b128(absent, rsrc, s + ml_at(c), 0, kSc1);
      }
  };
  Slots x, y;                                     // two looks under way, half a round trip apart
  for (int base = 0; base < nslots; base += SG * BATCH) {
    const auto load = [&](Slots& v) __attribute__((always_inline)) {
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
          const int s = (base + u * SG + sg) * step;
          v.ml[c][u] = __builtin_amdgcn_raw_buffer_load_b96(rsrc, s + ml_at(c), 0, kSc1);
          v.a[c][u] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, s + acc_at(c), 0, kSc1);
        }
      asm volatile("" ::: "memory");
    };
    const auto complete = [&](const Slots& v) __attribute__((always_inline)) {
      uint32_t most = 0;                          // kAbsent is the largest word
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
          most = max(max(max(most, v.ml[c][u].x), v.ml[c][u].y), ends_soon_or_absent(v.ml[c][u].z));
          most = max(max(most, v.a[c][u].x), v.a[c][u].y);
          most = max(max(most, v.a[c][u].z), v.a[c][u].w);
        }
      return !__any(most == kAbsent);
    };
    Slots z;
    load(x);
    if constexpr (ONCE) {
      if (!complete(x)) return false;
      z = x;
    } else {
      for (;;) {
        load(y);
        if (complete(x)) { z = x; break; }
        load(x);
        if (complete(y)) { z = y; break; }
        if ((tries += 2) >= ma.looks) return false;
      }
      if (base + SG * BATCH >= nslots) put_back();
    }
#pragma unroll
    for (int c = 0; c < C; ++c) {
      float mb = m_run[c], mv[BATCH];
#pragma unroll
      for (int u = 0; u < BATCH; ++u) {
        mv[u] = base + u * SG + sg < nslots ? __uint_as_float(z.ml[c][u].x) : kNegBig;
        mb = fmaxf(mb, mv[u]);
      }
      const float f0 = __builtin_amdgcn_exp2f(m_run[c] - mb);
      l_run[c] *= f0;
#pragma unroll
      for (int k = 0; k < 4; ++k) o_run[c][k] *= f0;
#pragma unroll
      for (int u = 0; u < BATCH; ++u) {
        const float f = __builtin_amdgcn_exp2f(mv[u] - mb);
        l_run[c] = __builtin_fmaf(__uint_as_float(z.ml[c][u].y), f, l_run[c]);
#pragma unroll
        for (int k = 0; k < 4; ++k) o_run[c][k] = __builtin_fmaf(__uint_as_float(z.a[c][u][k]), f, o_run[c][k]);
      }
      m_run[c] = mb;
    }
  }
  if constexpr (ONCE) {
    if (!take_block(ma, slot0, block0)) return false;
    put_back();
  }
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const float mm = head_max(m_run[c]);
    const float f = __builtin_amdgcn_exp2f(m_run[c] - mm);
    const float l = head_sum(l_run[c] * f);
    // the sums over the slot groups, the four channels turned into the four rows of lanes on the way
    float o[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) o[k] = o_run[c][k] * f;
    swap_rows(o[0], o[1]);
    swap_rows(o[2], o[3]);
    float lo = o[0] + o[1], hi = o[2] + o[3];
    swap_halves(lo, hi);
    float v = lo + hi;
    v += dpp_f32<0x124>(v);
    v += dpp_f32<0x128>(v);
    const int block = block0 + c * block_step;
    if ((lane & 12) == 0)
      ma.out[static_cast<int64_t>(item) * ma.g * kHeadDim + block * 16 + 4 * col + (lane >> 4)] = l > 0.f ? v / l : 0.f;
    if (lane == 0 && block % kBlocks == 0 && ma.lse != nullptr)
      ma.lse[static_cast<int64_t>(item) * ma.g + block / kBlocks] = l > 0.f ? (mm + __log2f(l)) * 0.6931471805599453f : -INFINITY;
  }
  // The look that was not needed is still on its way: its registers must not be used for anything before (that would wait for
  // it: 0.8 us).
  if constexpr (!ONCE) {
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
      for (int u = 0; u < BATCH; ++u) asm volatile("" ::"v"(x.a[c][u]), "v"(x.ml[c][u]), "v"(y.a[c][u]), "v"(y.ml[c][u]));
  }
  return true;
}

template <int NWV>
__device__ __forceinline__ int blocks_per_wave(const MergeArgs& ma) { return max(1, ma.g * kBlocks / ma.parts / NWV); }
// slots of a lane at a time: the same whoever merges, since the order of the sums depends on it
__device__ __forceinline__ int batch_of(int per_wave, int nslots) {
  return per_wave == 1 ? (nslots <= 32 ? 2 : 4) : per_wave == 2 ? (nslots <= 16 ? 1 : 2) : 1;
}

// lane -> a block of the heads whose partials this wavefront stores (heads wave, wave + NWV, ..; from 8 g on: none)
template <int NWV>
__device__ __forceinline__ int own_block() {
  const int lane = threadIdx.x & 63;
  return (static_cast<int>(threadIdx.x >> 6) + lane / kBlocks * NWV) * kBlocks + lane % kBlocks;
}

// A merging wavefront leaves its blocks to the chunks, except for what it need not be afraid of waiting for: the slots whose
// workgroups are through with their tiles.  The blocks, one bit each.
__device__ __forceinline__ uint64_t give_up(const MergeArgs& ma, int slot0, int nslots, int block0, int block_step, int n) {
  const int lane = threadIdx.x & 63;
  uint64_t blocks = 0;
  for (int k = 0; k < n; ++k) {
    const int block = block0 + k * block_step;
    blocks |= 1ull << block;
    for (int s = lane; s < nslots; s += 64) {
      if (clear_state(ma, slot0 + s, block, kGivenUp) & kEndsSoon) continue;
      for (int tries = 0; tries < kMostLooks; ++tries) {
        uint32_t most = 0;
        for (int w = 0; w < kStateWord; ++w)
          most = max(most, __hip_atomic_load(look_word(ma, slot0 + s, block, w), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        if (most != kAbsent) break;
      }
    }
  }
  if ((blocks >> lane) & 1)
    __hip_atomic_store(look_word(ma, slot0, lane, kHandOverWord), kReady, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  partial_stores_done();
  return blocks;
}

// A merging workgroup of NWV wavefronts (a chunk of tier kTierMerge): part ch.row0 of the item's blocks.  What comes back are
// the blocks of this wavefront, one bit each, that it has given up (merge_left).
template <int NWV>
__device__ __forceinline__ uint64_t merge_part(const MergeArgs& ma, const Chunk& ch) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int blocks = ma.g * kBlocks / ma.parts, block0 = ch.row0 * blocks + wave;
  if (wave >= blocks) return 0;
  // (merge_parts keeps a workgroup to four heads)
  const int per_wave = blocks_per_wave<NWV>(ma), batch = batch_of(per_wave, ch.nslots);
  bool done = true;
  switch (per_wave) {
    case 1:
      done = batch == 2 ? merge_blocks<1, 2, false>(ma, ch.item, ch.slot0, ch.nslots, block0, NWV)
                        : merge_blocks<1, 4, false>(ma, ch.item, ch.slot0, ch.nslots, block0, NWV);
      break;
    case 2:
      done = batch == 1 ? merge_blocks<2, 1, false>(ma, ch.item, ch.slot0, ch.nslots, block0, NWV)
                        : merge_blocks<2, 2, false>(ma, ch.item, ch.slot0, ch.nslots, block0, NWV);
      break;
    case 4: done = merge_blocks<4, 1, false>(ma, ch.item, ch.slot0, ch.nslots, block0, NWV); break;
    default:
      if constexpr (NWV < 8) done = merge_blocks<8, 1, false>(ma, ch.item, ch.slot0, ch.nslots, block0, NWV);
  }
  if (done) return 0;
  return give_up(ma, ch.slot0, ch.nslots, block0, NWV, per_wave);
}

// What a wavefront's heads' blocks have come to, of those whose partials it stores (store_partial), from the state words that it
// cleared a bit of when it was through with its tiles: the blocks that it has to look at, for merge_left.
template <int NWV>
__device__ __forceinline__ uint64_t blocks_left(const MergeArgs& ma, int slot0, uint32_t state) {
  if (!__any((state & kGivenUp) == 0)) return 0;
  partial_stores_done();
  uint32_t word = kAbsent;
  if ((state & kGivenUp) == 0)
    word = __hip_atomic_load(look_word(ma, slot0, own_block<NWV>(), kHandOverWord), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  uint64_t blocks = 0;
  for (uint64_t m = __ballot(word == kReady); m != 0; m &= m - 1) blocks |= 1ull << __builtin_amdgcn_readlane(own_block<NWV>(), __builtin_ctzll(m));
  return blocks;
}

// One look at each of these blocks; those whose words are all there are merged by whoever takes them first.
template <int NWV>
__device__ __forceinline__ void merge_left(const MergeArgs& ma, int item, int slot0, int nslots, uint64_t blocks) {
  const int batch = batch_of(blocks_per_wave<NWV>(ma), nslots);
  for (; blocks != 0; blocks &= blocks - 1) {
    const int block = __builtin_ctzll(blocks);
    if (batch == 1) merge_blocks<1, 1, true>(ma, item, slot0, nslots, block, 0);
    else if (batch == 2) merge_blocks<1, 2, true>(ma, item, slot0, nslots, block, 0);
    else merge_blocks<1, 4, true>(ma, item, slot0, nslots, block, 0);
  }
}

// LDS floats arrive_and_merge needs for NT threads (a flag, at most NT / 32 maxima and sums, four sums per thread)
__host__ __device__ constexpr int merge_lds_floats(int nt) { return 16 + 2 * (nt / 32) + nt * 4; }

}  // namespace merge
}  // namespace rdkv
