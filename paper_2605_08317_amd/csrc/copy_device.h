// The device side of a launch of small copies (CopyArgs), for the kernels that carry one along in workgroups of their own.
#pragma once
#include "rdkv_internal.h"

namespace rdkv {

constexpr int kCopyThreads = 256;
constexpr int kCopyRound = 4 * kCopyThreads;      // 16-byte units of a workgroup's round: four loads in flight per thread

struct __attribute__((packed, aligned(1))) Bytes16 { uint32_t v[4]; };

// 16 bytes past the caches (system scope), in one store: as four words the lanes' pieces cross PCIe one by one (70 us for 16 KB)
constexpr int kSystemScope = 17;
using uint4v = __attribute__((ext_vector_type(4))) unsigned;

// Workgroup b of the copies: every thread of a workgroup of kCopyThreads comes here.
__device__ __forceinline__ void copy_part(const CopyArgs& a, int b) {
  const int tid = threadIdx.x;
  int k = 0;
  for (int i = 1; i < a.n; ++i) k += b >= a.first[i];
  bool host = false;
  if (a.n > 0) {
    const CopySeg& s = a.seg[k];
    host = s.side != 0;
    const bool to_host = s.side == kDstHost;
    const int64_t n16 = s.bytes / 16, step = static_cast<int64_t>(a.first[k + 1] - a.first[k]) * kCopyRound;
    const Bytes16* src = static_cast<const Bytes16*>(s.src);
    Bytes16* dst = static_cast<Bytes16*>(s.dst);
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(s.dst, 0, static_cast<int>(n16 * 16), 0x00027000);   // (to_host: < 2 GiB)
    for (int64_t i0 = static_cast<int64_t>(b - a.first[k]) * kCopyRound + tid; i0 < n16; i0 += step) {
      Bytes16 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        v[u] = Bytes16{{s.fill[0], s.fill[1], s.fill[0], s.fill[1]}};
        if (s.src && i0 + u * kCopyThreads < n16) v[u] = src[i0 + u * kCopyThreads];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (i0 + u * kCopyThreads < n16) {
          if (to_host)
            __builtin_amdgcn_raw_buffer_store_b128(uint4v{v[u].v[0], v[u].v[1], v[u].v[2], v[u].v[3]}, rsrc,
                                                   static_cast<int>(i0 + u * kCopyThreads) * 16, 0, kSystemScope);
          else
            dst[i0 + u * kCopyThreads] = v[u];
        }
    }
    const int tail = static_cast<int>(s.bytes & 15);
    if (b == a.first[k] && tid < tail) {
      const int64_t at = 16 * n16 + tid;
      const uint8_t v = s.src ? static_cast<const uint8_t*>(s.src)[at] : static_cast<uint8_t>(s.fill[(at >> 2) & 1] >> (8 * (at & 3)));
      if (to_host) __hip_atomic_store(static_cast<uint8_t*>(s.dst) + at, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      else static_cast<uint8_t*>(s.dst)[at] = v;
    }
  }
  if (a.words && (host || a.n == 0)) {       // segments with a side in host memory come first: block b owns word b
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();                         // everything read from or written to the staging region is done
    if (tid == 0) __hip_atomic_store(a.words + b, a.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

}  // namespace rdkv
