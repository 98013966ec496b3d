// Small copies and fills of one call as a single launch: host tables out of pinned staging memory into device tables,
// counts back into pinned memory, parts of a cache's block copied and cleared.  A launch costs the host 2-3 us whatever it
// carries; as copies and memsets of the runtime the seven pieces of rdkv_pack took 25 us, and the two-way trip of the
// tier counts (a copy to pageable memory and a wait for the stream) 25 us beyond the kernels.
#include "rdkv_internal.h"

namespace rdkv {

namespace {

struct __attribute__((packed, aligned(1))) Bytes16 { uint32_t v[4]; };

__global__ __launch_bounds__(1024) void copy_kernel(CopyArgs a) {
  const int tid = threadIdx.x;
  for (int k = 0; k < a.n; ++k) {
    const CopySeg& s = a.seg[k];
    const int workers = s.host ? a.host_blocks : static_cast<int>(gridDim.x);
    if (static_cast<int>(blockIdx.x) >= workers) continue;
    const int64_t n16 = s.bytes / 16, step = static_cast<int64_t>(workers) * 1024;
    const Bytes16* src = static_cast<const Bytes16*>(s.src);
    Bytes16* dst = static_cast<Bytes16*>(s.dst);
    for (int64_t i0 = static_cast<int64_t>(blockIdx.x) * 1024 + tid; i0 < n16; i0 += 4 * step) {
      Bytes16 v[4];                        // four loads in flight
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        v[u] = Bytes16{{s.fill[0], s.fill[1], s.fill[0], s.fill[1]}};
        if (s.src && i0 + u * step < n16) v[u] = src[i0 + u * step];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (i0 + u * step < n16) dst[i0 + u * step] = v[u];
    }
    const int tail = static_cast<int>(s.bytes & 15);
    if (blockIdx.x == 0 && tid < tail) {
      const int64_t at = 16 * n16 + tid;
      static_cast<uint8_t*>(s.dst)[at] = s.src ? static_cast<const uint8_t*>(s.src)[at]
                                               : static_cast<uint8_t>(s.fill[(at >> 2) & 1] >> (8 * (at & 3)));
    }
  }
  if (a.words && static_cast<int>(blockIdx.x) < a.host_blocks) {
    __threadfence_system();                // everything read from or written to the staging region is done
    __syncthreads();
    if (tid == 0) __hip_atomic_store(a.words + blockIdx.x, a.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

}  // namespace

hipError_t launch_copy(const CopyArgs& a, hipStream_t st) {
  if (a.n == 0 && !a.words) return hipSuccess;
  int64_t most = 0;
  for (int k = 0; k < a.n; ++k)
    if (!a.seg[k].host && a.seg[k].bytes > most) most = a.seg[k].bytes;
  int64_t blocks = (most + 65535) / 65536;         // four rounds of 16 KB each
  if (blocks < a.host_blocks) blocks = a.host_blocks;
  if (blocks > 256) blocks = 256;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(copy_kernel, dim3(static_cast<unsigned>(blocks)), dim3(1024), 0, st, a);
  return hipGetLastError();
}

}  // namespace rdkv
