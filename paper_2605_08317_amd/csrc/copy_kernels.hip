// Small copies and fills of one call as a single launch: host tables out of pinned staging memory into device tables,
// counts back into pinned memory, parts of a cache's block copied and cleared.  A launch costs the host 2-3 us whatever it
// carries; as copies and memsets of the runtime the seven pieces of rdkv_pack took 25 us, and the two-way trip of the
// tier counts (a copy to pageable memory and a wait for the stream) 25 us beyond the kernels.
//
// What bounds it is latency: a read over PCIe takes 1.5 us, so every piece has workgroups of its own (pieces one after the
// other in each workgroup: 7 us a launch) and nothing is flushed: what goes to host memory goes past the caches, and a wait
// for the workgroup's own accesses stands in front of the completion word (a system-scope release writes back all of L2).
#include <algorithm>
#include <cstring>

#include "copy_device.h"

namespace rdkv {

namespace {

__global__ __launch_bounds__(kCopyThreads) void copy_kernel(CopyArgs a) { copy_part(a, blockIdx.x); }

// Bytes that come with the launch: of a graph's node, which keeps its arguments.
struct ValueArgs {
  uint8_t* dst;
  int32_t bytes;
  uint8_t data[3072];                  // (a launch carries up to 4 KB of arguments)
};
__global__ __launch_bounds__(kCopyThreads) void copy_value_kernel(ValueArgs a) {
  for (int i = threadIdx.x; i < a.bytes; i += kCopyThreads) a.dst[i] = a.data[i];
}

}  // namespace

void plan_copy(CopyArgs& a) {
  // segments with a host side share the completion words
  int n_host = 0;
  int64_t host_bytes = 0;
  for (int k = 0; k < a.n; ++k)
    if (a.seg[k].side != 0) { ++n_host; host_bytes += a.seg[k].bytes; }
  const int64_t least = kCopyRound * 16;
  int64_t host_part = least;
  if (n_host > 0) host_part = std::max(least, (host_bytes + kStageWords - n_host - 1) / (kStageWords - n_host));
  int at = 0;
  for (int k = 0; k < a.n; ++k) {
    const CopySeg& s = a.seg[k];
    a.first[k] = at;
    const int64_t part = s.side != 0 ? host_part : least;
    at += static_cast<int>(std::min<int64_t>(std::max<int64_t>((s.bytes + part - 1) / part, 1), 2048));
    if (s.side != 0) a.host_blocks = at;
  }
  a.first[a.n] = at;
  if (a.n == 0) a.host_blocks = 1;
}

hipError_t launch_copy(const CopyArgs& a, hipStream_t st) {
  if (a.n == 0 && !a.words) return hipSuccess;
  const int blocks = a.n == 0 ? 1 : a.first[a.n];
  hipLaunchKernelGGL(copy_kernel, dim3(static_cast<unsigned>(blocks)), dim3(kCopyThreads), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_copy_by_value(const CopyArgs& a, hipStream_t st) {
  for (int k = 0; k < a.n; ++k)
    if (a.seg[k].side != kSrcHost) return hipErrorStreamCaptureUnsupported;
  for (int k = 0; k < a.n; ++k) {
    const CopySeg& s = a.seg[k];
    ValueArgs v{};
    for (int64_t at = 0; at < s.bytes; at += v.bytes) {
      v.dst = static_cast<uint8_t*>(s.dst) + at;
      v.bytes = static_cast<int32_t>(std::min<int64_t>(s.bytes - at, sizeof(v.data)));
      std::memcpy(v.data, static_cast<const uint8_t*>(s.src) + at, v.bytes);
      hipLaunchKernelGGL(copy_value_kernel, dim3(1), dim3(kCopyThreads), 0, st, v);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
  }
  return hipSuccess;
}

}  // namespace rdkv
