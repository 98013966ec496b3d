// The kernels over row-major bf16 rows (decode_rows.h): the uncompressed path, and the 16-bit tier of a token-wise cache
// whose launch is too large for the quantized tiers' kernel to take it along.
#include "decode_rows.h"

namespace rdkv {

namespace {

using namespace tile;

constexpr int kRowsWaves = 4;
constexpr int kRowsWG = kRowsWaves * 64;

// The merge inside the launch.  The caller's workspace holds no counter that starts at zero, and nothing else outlives the call, so
// chunks announce themselves by the launch's tag, in the item's own output rows, which hold whatever they held before (two words a
// chunk, NaNs that neither a result nor an earlier launch leaves).  A chunk stores its partial, its tag once that has landed, and
// looks at all of the item's tags once its own has: the chunk whose tag lands last finds all of them, or finds that another one
// has, and has begun to write the rows.  Several may find all of them; they write the same bits.  Nothing waits for anybody, and the
// merge leaves no tag behind (a replayed launch has the same one).
// What bounds it is four round trips to memory: partial, tag, tags, partials; and with many partials one compute unit's reading of
// them (dense_together in rdkv_api.hip has the line and what was measured on both sides of it).
template <int HS>
__device__ __forceinline__ void merge_tagged(const DenseArgs& a, int item, int slot0, int split, int n, int g, uint8_t* smem) {
  const int tid = threadIdx.x, lane = tid & 63;
  uint32_t* tags = reinterpret_cast<uint32_t*>(a.out + static_cast<int64_t>(item) * g * kHeadDim);
  merge::partial_stores_done();
  __syncthreads();
  if (n > 1) {
    int* s_all = reinterpret_cast<int*>(smem);
    if (tid < 64) {
      if (lane < 2) __hip_atomic_store(tags + 2 * split + lane, a.tag[lane & 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      merge::partial_stores_done();
      bool there = true;
      if (lane < n) {
        const uint32_t t0 = __hip_atomic_load(tags + 2 * lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t t1 = __hip_atomic_load(tags + 2 * lane + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        there = t0 == a.tag[0] && t1 == a.tag[1];
      }
      const bool all = __all(there);
      if (tid == 0) *s_all = all;
    }
    __syncthreads();
    if (*s_all == 0) return;
    __syncthreads();                    // the merge uses that memory
  }
  const MergeArgs ma{a.part_acc, a.part_ml, nullptr, a.out, a.lse, g, 0, 0};
  float* s = reinterpret_cast<float*>(smem);
  // (one round trip for all that dense_together lets come here, and not many more loads than there are partials: with sixteen a thread
  // for two heads of up to 32, the launch took from a graph what two do or 0.2 us more; 2 x 2K rows 8.53, 8.48 -> 7.85 us, 16 x 4K with
  // 62 MB 17.2, 17.8 -> 16.75)
  if constexpr (HS == 2) {
    if (n <= 8) merge::merge_item<kRowsWG, 8, 8, true>(ma, item, slot0, n, s);
    else merge::merge_item<kRowsWG, 8, 16, true>(ma, item, slot0, n, s);
  } else if (g == 4) {
    if (n <= 16) merge::merge_item<kRowsWG, 4, 8, true>(ma, item, slot0, n, s);
    else merge::merge_item<kRowsWG, 4, 16, true>(ma, item, slot0, n, s);
  } else if (g == 2) {
    if (n <= 32) merge::merge_item<kRowsWG, 2, 8, true>(ma, item, slot0, n, s);
    else merge::merge_item<kRowsWG, 2, 16, true>(ma, item, slot0, n, s);
  } else {
    merge::merge_item<kRowsWG, 1, 8, true>(ma, item, slot0, n, s);
  }
}

// TOGETHER: it merges its own partials (an instantiation of its own, so that the launch that leaves them to another is not slower for the
// merge's code and registers: one sequence of 20K rows, four heads, 13.56 -> 14.04 us a call).
template <int HS, bool TOGETHER>
__global__ __launch_bounds__(kRowsWG, 2) void decode_dense_mfma_kernel(DenseArgs a) {
  extern __shared__ __align__(16) uint8_t smem[];
  const int split = blockIdx.x, head = blockIdx.y, sl = blockIdx.z;
  const int T = a.T[sl];
  const int row0 = split * a.chunk_rows;
  const int g = a.hq / a.hkv;
  if (row0 >= T) {
    if (TOGETHER && split == 0) {       // no rows at all, and no merge launch
      const int64_t qh0 = static_cast<int64_t>(a.seq_base + sl) * a.hq + head * g;
      for (int i = threadIdx.x; i < g * kHeadDim; i += kRowsWG) a.out[qh0 * kHeadDim + i] = 0.f;
      if (a.lse != nullptr && static_cast<int>(threadIdx.x) < g) a.lse[qh0 + threadIdx.x] = -INFINITY;
    }
    return;
  }
  const int rows = min(a.chunk_rows, T - row0);
  const int64_t first = a.row_off[sl] + static_cast<int64_t>(head) * T + row0;
  const uint8_t* kd = reinterpret_cast<const uint8_t*>(a.K) + first * (kHeadDim * 2);
  const uint8_t* vd = reinterpret_cast<const uint8_t*>(a.V) + first * (kHeadDim * 2);
  const int seq = a.seq_base + sl;
  const uint16_t* q = a.q + (static_cast<int64_t>(seq) * a.hq + head * g) * kHeadDim;
  const int64_t slot = (static_cast<int64_t>(sl) * a.hkv + head) * a.max_splits + split;
  process_rows_mfma<HS, false, kRowsWaves, false, TOGETHER>(kd, vd, rows, g, q, smem, a.part_acc + slot * g * kHeadDim,
                                                            a.part_ml + slot * g * 2, nullptr, nullptr);
  if constexpr (TOGETHER)
    merge_tagged<HS>(a, seq * a.hkv + head, static_cast<int>(slot) - split, split, (T + a.chunk_rows - 1) / a.chunk_rows, g, smem);
}

template <int HS>
__global__ __launch_bounds__(kRowsWG, 2) void decode_tiered_mfma_kernel(const Chunk* __restrict__ chunks,
                                                                       const uint8_t* __restrict__ arena,
                                                                       const uint16_t* __restrict__ q, int g, MergeArgs ma) {
  extern __shared__ __align__(16) uint8_t smem[];
  const Chunk ch = chunks[blockIdx.x];
  const uint16_t* qp = q + static_cast<int64_t>(ch.item) * g * kHeadDim;     // item = sequence x KV head
  const ChunkOut co{ch.item, ch.slot, ch.slot0, ch.nslots};
  process_rows_mfma<HS, true, kRowsWaves>(arena + ch.k_data, arena + ch.v_data, ch.rows, g, qp, smem,
                              ma.part_acc + static_cast<int64_t>(ch.slot) * g * kHeadDim,
                              ma.part_ml + static_cast<int64_t>(ch.slot) * g * 2, &ma, &co);
}

}  // namespace

template <int HS, bool TOGETHER>
static hipError_t launch_dense(const DenseArgs& a, int n_seqs, hipStream_t st) {
  const size_t lds = rows_lds_bytes<HS, kRowsWaves>();
  const hipError_t e = RDKV_ALLOW_LDS((decode_dense_mfma_kernel<HS, TOGETHER>), lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((decode_dense_mfma_kernel<HS, TOGETHER>), dim3(a.max_splits, a.hkv, n_seqs), dim3(kRowsWG), lds, st, a);
  return hipGetLastError();
}
hipError_t launch_decode_dense_split(const DenseArgs& a, int g, int n_seqs, hipStream_t st) {
  const bool together = a.tag[0] != 0;
  if (g > 4) return together ? launch_dense<2, true>(a, n_seqs, st) : launch_dense<2, false>(a, n_seqs, st);
  return together ? launch_dense<1, true>(a, n_seqs, st) : launch_dense<1, false>(a, n_seqs, st);
}

hipError_t launch_decode_tiered_split(const Chunk* chunks, int n_chunks, const uint8_t* arena, const uint16_t* q,
                                      const MergeArgs& ma, hipStream_t st) {
  if (n_chunks == 0) return hipSuccess;
  dim3 grid(n_chunks), block(kRowsWG);
  if (ma.g > 4) {
    const size_t lds = rows_lds_bytes<2, kRowsWaves>();
    hipError_t e = RDKV_ALLOW_LDS((decode_tiered_mfma_kernel<2>), lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(decode_tiered_mfma_kernel<2>, grid, block, lds, st, chunks, arena, q, ma.g, ma);
  } else {
    const size_t lds = rows_lds_bytes<1, kRowsWaves>();
    hipError_t e = RDKV_ALLOW_LDS((decode_tiered_mfma_kernel<1>), lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(decode_tiered_mfma_kernel<1>, grid, block, lds, st, chunks, arena, q, ma.g, ma);
  }
  return hipGetLastError();
}

}  // namespace rdkv
