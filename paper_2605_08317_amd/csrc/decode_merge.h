// Log-sum-exp merge of the split partials of a decode step (the last step of Eq. 7's evaluation as a split-K
// flash-decode) inside the decode kernels themselves: every workgroup stores its chunk's partial result, announces
// it on the item's arrival counter, and the workgroup that arrives last merges all partials of the item and writes
// the output rows.  One launch per decode step instead of a split launch and a merge launch.
//
// Memory ordering across the chip's eight L2 caches: partials are written and read with agent-scope accesses (they
// go through to memory instead of staying in one XCD's L2), every thread waits for its stores to drain before the
// workgroup's barrier, and one thread then bumps the counter with an agent-scope atomic.  The merging workgroup resets the
// counter, so a cache's workspace is ready for the next step on the same stream.  The merge has a fixed summation
// order (slot order), so results do not depend on which workgroup happens to arrive last.
#pragma once
#include "rdkv_internal.h"

namespace rdkv {

struct MergeArgs {
  float* part_acc;     // [slots][g][128] unnormalised partial outputs
  float* part_ml;      // [slots][g][2]   running maximum (log2 domain) and sum of each partial
  int32_t* arrive;     // [items] arrival counters, zero between steps
  float* out;          // [batch][hq][128]
  float* lse;          // [batch][hq] or null
  int32_t g;           // query heads per KV head: item i (sequence x KV head) owns output rows i g .. i g + g - 1
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

__device__ __forceinline__ void store_agent(float* p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
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
constexpr int kSc1 = 16;                  // cache policy of the buffer accesses: agent scope

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
  using uint4v = __attribute__((ext_vector_type(4))) unsigned;
  using uint2v = __attribute__((ext_vector_type(2))) unsigned;
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

// LDS floats arrive_and_merge needs for NT threads (the flag, SG * G <= NT / 32 maxima and sums, four sums per thread)
__host__ __device__ constexpr int merge_lds_floats(int nt) { return 16 + 2 * (nt / 32) + nt * 4; }

}  // namespace merge
}  // namespace rdkv
