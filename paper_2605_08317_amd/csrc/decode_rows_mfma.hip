// The kernels over row-major bf16 rows (decode_rows.h): the uncompressed path, and the 16-bit tier of a token-wise cache
// whose launch is too large for the quantized tiers' kernel to take it along.
#include "decode_rows.h"

namespace rdkv {

namespace {

using namespace tile;

constexpr int kRowsWaves = 4;
constexpr int kRowsWG = kRowsWaves * 64;

template <int HS>
__global__ __launch_bounds__(kRowsWG, 2) void decode_dense_mfma_kernel(DenseArgs a) {
  extern __shared__ __align__(16) uint8_t smem[];
  const int split = blockIdx.x, head = blockIdx.y, sl = blockIdx.z;
  const int T = a.T[sl];
  const int row0 = split * a.chunk_rows;
  if (row0 >= T) return;
  const int g = a.hq / a.hkv;
  const int rows = min(a.chunk_rows, T - row0);
  const int64_t first = a.row_off[sl] + static_cast<int64_t>(head) * T + row0;
  const uint8_t* kd = reinterpret_cast<const uint8_t*>(a.K) + first * (kHeadDim * 2);
  const uint8_t* vd = reinterpret_cast<const uint8_t*>(a.V) + first * (kHeadDim * 2);
  const int seq = a.seq_base + sl;
  const uint16_t* q = a.q + (static_cast<int64_t>(seq) * a.hq + head * g) * kHeadDim;
  const int64_t slot = (static_cast<int64_t>(sl) * a.hkv + head) * a.max_splits + split;
  process_rows_mfma<HS, false, kRowsWaves>(kd, vd, rows, g, q, smem, a.part_acc + slot * g * kHeadDim, a.part_ml + slot * g * 2,
                               nullptr, nullptr);
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

hipError_t launch_decode_dense_split(const DenseArgs& a, int g, int n_seqs, hipStream_t st) {
  dim3 grid(a.max_splits, a.hkv, n_seqs), block(kRowsWG);
  if (g > 4) {
    const size_t lds = rows_lds_bytes<2, kRowsWaves>();
    hipError_t e = RDKV_ALLOW_LDS((decode_dense_mfma_kernel<2>), lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(decode_dense_mfma_kernel<2>, grid, block, lds, st, a);
  } else {
    const size_t lds = rows_lds_bytes<1, kRowsWaves>();
    hipError_t e = RDKV_ALLOW_LDS((decode_dense_mfma_kernel<1>), lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(decode_dense_mfma_kernel<1>, grid, block, lds, st, a);
  }
  return hipGetLastError();
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
