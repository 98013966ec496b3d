// Host side of librdkv: argument validation, planning (segment table, split
// schedule) and kernel launches behind the C ABI of include/rdkv.h.
#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <initializer_list>
#include <mutex>
#include <new>
#include <thread>
#include <utility>

#include "decode_merge.h"
#include "dense_plan.h"
#include "rdkv_internal.h"

namespace rdkv {
hipError_t launch_tier_count(const uint8_t* bits, const Batch& batch, int32_t* blk_counts, int max_T, hipStream_t st);
hipError_t launch_tier_scatter(const uint8_t* bits, const Batch& batch, const int32_t* blk_counts, int32_t* tier_idx,
                               const PlanArgs& plan, int max_T, const CopyArgs& copy, hipStream_t st);
hipError_t launch_quant_pack(const uint16_t* K, const uint16_t* V, const int32_t* tier_idx, int32_t* tier_idx_out,
                             const PlanArgs& plan, const Batch& batch, uint8_t* arena, int max_tiles,
                             uint32_t* k_range, int row_wide, const CopyArgs& copy, hipStream_t st);
size_t weights_scratch_floats(int64_t n_tiles, int64_t n_items, int64_t total_tokens, int R, bool want_ch);
hipError_t launch_weights(const rdkv_config& cfg, const Batch& batch, int64_t n_tiles, int64_t n_items, int64_t total_tokens,
                          int max_T, const uint16_t* K, const uint16_t* Q_obs, float* w_tok, float* w_ch,
                          float* scratch, const float** raw, hipStream_t st);
size_t allocate_scratch_bytes(int n_items, int max_U);
bool allocate_needs_order(int n_items, int max_U);
int allocate_short_units();
hipError_t launch_allocate(const float* raw, int pool, float* w, const Batch& batch, int max_U, const int32_t* d_order, int n_long,
                           int max_short, int n_hull, const int* hull_tiers,
                           const double* hull_r, double need_frac, int max_iters, uint8_t* bits, double* lam_out,
                           int32_t* iters_out, int32_t* blk_counts, const CountPost& post, void* scratch, hipStream_t st);
hipError_t launch_allocate_channels(const float* w_ch, const Batch& batch, const int32_t* blk_counts, double rk, int n_hull,
                                    const int* hull_tiers,
                                    const double* hull_r, double need_frac, int max_iters, uint8_t* bits_ch,
                                    double* lam_out, int32_t* iters_out, const CountPost& post, hipStream_t st);
hipError_t launch_calibrate(const uint16_t* K, const uint16_t* V, const int64_t* item_row_off, const int32_t* item_T,
                            int n_items, int max_T, bool k_channelwise, bool k_whole_channel, bool row_wide,
                            double* acc_k, double* acc_v, uint32_t* range, hipStream_t st);
}  // namespace rdkv

using namespace rdkv;


namespace {

thread_local std::string g_err;

rdkv_status fail(rdkv_status s, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  g_err = buf;
  return s;
}

#define RDKV_HIP(expr)                                                                      \
  do {                                                                                      \
    hipError_t e_ = (expr);                                                                 \
    if (e_ != hipSuccess) return fail(RDKV_ERR_HIP, "%s: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

int64_t round_up(int64_t x, int64_t a) { return (x + a - 1) / a * a; }

// ---- optional event bracketing of the main kernels ----------------------------------
struct KernelTiming {
  std::mutex mu;
  bool enabled = false;
  std::vector<std::pair<hipEvent_t, hipEvent_t>> ev[RDKV_TIME_KINDS];
  std::vector<hipEvent_t> pool;
  hipEvent_t get() {
    if (!pool.empty()) { hipEvent_t e = pool.back(); pool.pop_back(); return e; }
    hipEvent_t e = nullptr;
    return hipEventCreate(&e) == hipSuccess ? e : nullptr;
  }
};
KernelTiming g_timing;

constexpr int kMaxDevices = 64;

// Scratch of calls without allocator hooks: blocks that outlive the call, one pool per device.  (hipFreeAsync waits for the
// stream when the block was handed out again before its previous hipFreeAsync had come up on it: the second of two staged
// calls behind a quarter of a second of queued work took 242 ms to return, now 0.02.)
// A block given back carries an event of its last stream; it goes out again to that stream, or to another one once the event
// has passed.  At most kBytes per device; what does not fit comes from the runtime's pool and may wait.  Blocks that were not
// used for a while go back when a cache is freed, which waits for the device anyway.
class ScratchPool {
  struct Block { void* p; size_t bytes; hipEvent_t ev; hipStream_t st; bool idle; uint64_t used; };
  std::mutex mu_;
  std::vector<Block> blocks_;
  size_t total_ = 0;
  uint64_t calls_ = 0;
  static constexpr size_t kBytes = static_cast<size_t>(512) << 20;
  static constexpr uint64_t kKeepCalls = 64;
  // sizes in quarter steps of a power of two, so that a program's largest call leaves few blocks behind
  static size_t rounded(size_t bytes) {
    size_t step = static_cast<size_t>(64) << 10;
    while (8 * step <= bytes) step *= 2;
    return (bytes + step - 1) / step * step;
  }

 public:
  void* get(size_t bytes, hipStream_t st) {
    std::lock_guard<std::mutex> lk(mu_);
    ++calls_;
    Block* best = nullptr;
    for (Block& b : blocks_)
      if (b.idle && b.bytes >= bytes && (!best || b.bytes < best->bytes) && (b.st == st || hipEventQuery(b.ev) == hipSuccess)) best = &b;
    if (best) {
      if (hipEventQuery(best->ev) != hipSuccess && hipStreamWaitEvent(st, best->ev, 0) != hipSuccess) return nullptr;
      best->idle = false;
      best->used = calls_;
      return best->p;
    }
    Block b{nullptr, rounded(bytes), nullptr, st, false, calls_};
    if (total_ + b.bytes > kBytes) return nullptr;
    if (hipEventCreateWithFlags(&b.ev, hipEventDisableTiming) != hipSuccess) return nullptr;
    if (hipMallocAsync(&b.p, b.bytes, st) != hipSuccess) {      // (hipMalloc would end another thread's graph capture)
      (void)hipEventDestroy(b.ev);
      return nullptr;
    }
    blocks_.push_back(b);
    total_ += b.bytes;
    return b.p;
  }
  bool put(void* p, hipStream_t st) {      // false: not of this pool
    std::lock_guard<std::mutex> lk(mu_);
    for (Block& b : blocks_)
      if (b.p == p) {
        if (hipEventRecord(b.ev, st) != hipSuccess) (void)hipStreamSynchronize(st);
        b.st = st;
        b.idle = true;
        return true;
      }
    return false;
  }
  void give_back() {
    std::lock_guard<std::mutex> lk(mu_);
    for (size_t k = 0; k < blocks_.size();) {
      Block& b = blocks_[k];
      if (!b.idle || calls_ - b.used < kKeepCalls || hipEventQuery(b.ev) != hipSuccess) { ++k; continue; }
      (void)hipFreeAsync(b.p, nullptr);
      (void)hipEventDestroy(b.ev);
      total_ -= b.bytes;
      b = blocks_.back();
      blocks_.pop_back();
    }
  }
};
ScratchPool g_scratch_pool[kMaxDevices];
ScratchPool* scratch_pool() {
  int dev = -1;
  return hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < kMaxDevices ? &g_scratch_pool[dev] : nullptr;
}

// Device memory of the library.  What a cache owns lives until rdkv_cache_free and comes from alloc() / hipMalloc.
// Scratch of a single call is released when the call returns, while its kernels may still be queued: the release is
// stream-ordered (the caller's hooks must behave like a stream-ordered caching allocator on the call's stream; without
// hooks the pool above, or hipMallocAsync / hipFreeAsync on that stream when it is under capture).
struct Allocator {
  rdkv_alloc_fn alloc = nullptr;
  rdkv_free_fn free_ = nullptr;
  void* user = nullptr;
  void* get(size_t bytes) const {
    if (bytes == 0) bytes = 16;
    if (alloc) return alloc(bytes, user);
    void* p = nullptr;
    return hipMalloc(&p, bytes) == hipSuccess ? p : nullptr;
  }
  void put(void* p) const {
    if (!p) return;
    if (free_) free_(p, user); else (void)hipFree(p);
  }
  void* get_scratch(size_t bytes, hipStream_t st) const {
    if (bytes == 0) bytes = 16;
    if (alloc) return alloc(bytes, user);
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cap) == hipSuccess && cap == hipStreamCaptureStatusNone)
      if (ScratchPool* pool = scratch_pool())
        if (void* p = pool->get(bytes, st)) return p;
    void* p = nullptr;
    return hipMallocAsync(&p, bytes, st) == hipSuccess ? p : nullptr;
  }
  void put_scratch(void* p, hipStream_t st) const {
    if (!p) return;
    if (free_) { free_(p, user); return; }
    ScratchPool* pool = scratch_pool();
    if (!pool || !pool->put(p, st)) (void)hipFreeAsync(p, st);
  }
};

// Device scratch that is released (stream-ordered) when the call returns.  reserve() takes one allocation up front
// that the following get() calls are carved from; requests that do not fit fall back to allocations of their own.
struct Temp {
  const Allocator& al;
  hipStream_t st;
  std::vector<void*> ptrs;
  uint8_t* slab = nullptr;
  size_t slab_bytes = 0, used = 0;
  Temp(const Allocator& a, hipStream_t s) : al(a), st(s) {}
  ~Temp() { for (void* p : ptrs) al.put_scratch(p, st); }
  static size_t padded(size_t bytes) { return (std::max<size_t>(bytes, 16) + 255) / 256 * 256; }
  void reserve(std::initializer_list<size_t> sizes) {
    size_t total = 0;
    for (size_t b : sizes) total += padded(b);
    slab = static_cast<uint8_t*>(al.get_scratch(total, st));
    if (slab) {
      ptrs.push_back(slab);
      slab_bytes = total;
    }
  }
  template <typename T>
  T* get(size_t n) {
    const size_t b = padded(n * sizeof(T));
    if (slab && used + b <= slab_bytes) {
      T* p = reinterpret_cast<T*>(slab + used);
      used += b;
      return p;
    }
    void* p = al.get_scratch(n * sizeof(T), st);
    if (p) ptrs.push_back(p);
    return static_cast<T*>(p);
  }
};

// Host tables of a call, and the counts it reads back, travel through a ring of pinned memory (one per device) that
// kernels read and write directly (launch_copy): no copy of the runtime, no event, no wait for the stream.  A region starts
// with completion words that the kernel sets to the region's number when it is done with it; the ring's bytes are reused
// once it has.
constexpr size_t kStageHead = kStageWords * sizeof(uint32_t);

struct StageRegion {
  uint8_t* data = nullptr;        // pinned: what the host fills (or reads)
  uint32_t* words = nullptr;
  uint32_t seq = 0;
  void* own = nullptr;            // not of the ring: an allocation of its own
  bool recorded = false;          // the stream is under capture: `own` is ordinary memory that no kernel ever sees
  bool done() const {
    for (int i = 0; i < kStageWords; ++i)
      if (__atomic_load_n(words + i, __ATOMIC_ACQUIRE) != seq) return false;
    return true;
  }
  void mark_done() const {        // no kernel will
    for (int i = 0; i < kStageWords; ++i) __atomic_store_n(words + i, seq, __ATOMIC_RELEASE);
  }
};

// Spins until the region's kernel is done.  The stream is asked now and then, so that a failed launch or a fault ends the
// wait.
hipError_t stage_wait(const StageRegion& r, hipStream_t st) {
  for (uint32_t spins = 1;; ++spins) {
    if (r.done()) return hipSuccess;
#if defined(__x86_64__)
    __builtin_ia32_pause();
#endif
    if ((spins & 0x3FFF) == 0) {
      const hipError_t e = hipStreamQuery(st);
      if (e == hipErrorNotReady) continue;
      if (e == hipSuccess && r.done()) return hipSuccess;
      r.mark_done();
      return e != hipSuccess ? e : hipErrorUnknown;
    }
  }
}

class Staging {
  struct Live { size_t begin, end; StageRegion r; bool held; };
  std::mutex mu_;
  uint8_t* base_ = nullptr;
  size_t head_ = 0;
  uint32_t seq_ = 0;
  std::deque<Live> live_;          // regions whose kernel may not have run yet, or that the host still reads
  static constexpr size_t kBytes = static_cast<size_t>(2) << 20;

 public:
  // A region of `bytes`; `held`: the host reads it back and calls release().
  hipError_t acquire(size_t bytes, bool held, StageRegion* out) {
    std::unique_lock<std::mutex> lk(mu_);
    if (!base_) {
      void* p = nullptr;
      const hipError_t e = hipHostMalloc(&p, kBytes, hipHostMallocDefault);
      if (e != hipSuccess) return e;
      base_ = static_cast<uint8_t*>(p);
    }
    const size_t need = (kStageHead + bytes + 255) / 256 * 256;
    StageRegion r;
    r.seq = ++seq_ ? seq_ : ++seq_;
    uint8_t* p = nullptr;
    if (need > kBytes / 2) {        // larger than the ring: memory of its own
      const hipError_t e = hipHostMalloc(&r.own, need, hipHostMallocDefault);
      if (e != hipSuccess) return e;
      p = static_cast<uint8_t*>(r.own);
    } else {
      if (head_ + need > kBytes) head_ = 0;     // wrap: the bytes up to the end of the ring are skipped
      for (size_t k = 0; k < live_.size();) {   // regions on the bytes about to be overwritten
        const Live& l = live_[k];
        if (l.begin >= head_ + need || l.end <= head_) { ++k; continue; }
        if (l.held && !l.r.done()) {            // another thread waits for it: go on behind it
          head_ = l.end + need > kBytes ? 0 : l.end;
          k = 0;
          continue;
        }
        wait_for(l.r);
        if (l.held) {                           // read back within microseconds by the thread that holds it
          lk.unlock();
          std::this_thread::yield();
          lk.lock();
          k = 0;
          continue;
        }
        live_.erase(live_.begin() + static_cast<std::ptrdiff_t>(k));
      }
      while (!live_.empty() && !live_.front().held && live_.front().r.done()) live_.pop_front();
      p = base_ + head_;
    }
    r.words = reinterpret_cast<uint32_t*>(p);
    r.data = p + kStageHead;
    for (int i = 0; i < kStageWords; ++i) __atomic_store_n(r.words + i, 0u, __ATOMIC_RELAXED);
    if (!r.own) {
      live_.push_back(Live{head_, head_ + need, r, held});
      head_ += need;
    }
    *out = r;
    return hipSuccess;
  }
  // The host is done with a held region.
  void release(const StageRegion& r) {
    std::lock_guard<std::mutex> lk(mu_);
    for (Live& l : live_)
      if (l.r.words == r.words && l.r.seq == r.seq) l.held = false;
  }

 private:
  static void wait_for(const StageRegion& r) {
    for (uint32_t spins = 1; !r.done(); ++spins) {
#if defined(__x86_64__)
      __builtin_ia32_pause();
#endif
      if ((spins & 0xFFFFFF) == 0 && hipDeviceSynchronize() != hipSuccess) return;   // the device is lost
    }
  }
};
Staging g_staging[kMaxDevices];

// A region for a launch on `st`.  Under capture the bytes travel in the recorded launches' arguments: a replay comes when
// a region of the ring is long somebody else's.
hipError_t stage_acquire(size_t bytes, bool held, hipStream_t st, StageRegion* out, int* device) {
  hipError_t e = hipGetDevice(device);
  if (e != hipSuccess) return e;
  if (*device < 0 || *device >= kMaxDevices) return hipErrorInvalidDevice;
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (!held) e = hipStreamIsCapturing(st, &cap);          // (the calls that wait have asked: refuse_capture)
  if (e != hipSuccess) return e;
  if (cap == hipStreamCaptureStatusNone) return g_staging[*device].acquire(bytes, held, out);
  StageRegion r;
  r.recorded = true;
  r.own = std::malloc(std::max<size_t>(bytes, 1));
  if (!r.own) return hipErrorOutOfMemory;
  r.data = static_cast<uint8_t*>(r.own);
  *out = r;
  return hipSuccess;
}

// Launches a copy to or from a region.  `last`: the region's only launch and not read by the host; memory that is not of
// the ring is given back then (after the kernel; the ring looks after itself).  `launch`: the kernel that takes the planned copy
// along (not under capture).
template <class Launch>
hipError_t stage_launch(CopyArgs& a, const StageRegion& r, bool last, hipStream_t st, Launch&& launch) {
  if (r.recorded) {
    const hipError_t e = launch_copy_by_value(a, st);
    std::free(r.own);
    return e;
  }
  plan_copy(a);
  a.words = r.words;
  a.seq = r.seq;
  for (int i = a.host_blocks; i < kStageWords; ++i) __atomic_store_n(r.words + i, r.seq, __ATOMIC_RELAXED);   // nobody's
  hipError_t e = launch(a);
  if (e != hipSuccess) r.mark_done();
  if (last && r.own) {
    if (e == hipSuccess) e = stage_wait(r, st);
    (void)hipHostFree(r.own);
  }
  return e;
}
hipError_t stage_launch(CopyArgs& a, const StageRegion& r, bool last, hipStream_t st) {
  return stage_launch(a, r, last, st, [&](const CopyArgs& c) { return launch_copy(c, st); });
}

// For the calls that wait for the stream: refuses a stream under capture before anything is recorded.
rdkv_status refuse_capture(hipStream_t st) {
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  RDKV_HIP(hipStreamIsCapturing(st, &cap));
  if (cap == hipStreamCaptureStatusNone) return RDKV_OK;
  return fail(RDKV_ERR_HIP, "the call waits for the stream, which is under capture: %s", hipGetErrorString(hipErrorStreamCaptureUnsupported));
}

// Launches a copy, waits for it -- and so for everything queued on the stream before it -- and hands the region to `read`.
// (A copy to pageable memory and a wait for the stream: 25-35 us beyond the work; so 3-5.)
template <class Read, class Launch>
hipError_t stage_round_trip(CopyArgs& a, int device, const StageRegion& r, hipStream_t st, Read&& read, Launch&& launch) {
  hipError_t e = stage_launch(a, r, false, st, launch);
  if (e == hipSuccess) e = stage_wait(r, st);
  if (e == hipSuccess) read();
  g_staging[device].release(r);
  if (r.own) (void)hipHostFree(r.own);
  return e;
}
template <class Read>
hipError_t stage_round_trip(CopyArgs& a, int device, const StageRegion& r, hipStream_t st, Read&& read) {
  return stage_round_trip(a, device, r, st, read, [&](const CopyArgs& c) { return launch_copy(c, st); });
}

// Words that the search's kernels post for the host (CountPost).
class Posted {
  StageRegion r_;
  int dev_ = 0;
  hipStream_t st_ = nullptr;
  uint64_t* words_ = nullptr;
  int64_t n_ = 0, n_counts_ = 0;

 public:
  Posted() = default;
  Posted(const Posted&) = delete;
  Posted& operator=(const Posted&) = delete;
  // (a call that failed in between: what was launched may still post)
  ~Posted() {
    if (words_) {
      (void)hipStreamSynchronize(st_);
      give_back();
    }
  }
  hipError_t open(int64_t n_items, bool channels, hipStream_t st) {
    n_counts_ = 4 * n_items;
    n_ = n_counts_ + (channels ? 16 * n_items : 0);
    const hipError_t e = stage_acquire(static_cast<size_t>(n_) * sizeof(uint64_t), true, st, &r_, &dev_);
    if (e != hipSuccess) return e;
    st_ = st;
    words_ = reinterpret_cast<uint64_t*>(r_.data);
    for (int64_t i = 0; i < n_; ++i) __atomic_store_n(words_ + i, uint64_t{0}, __ATOMIC_RELAXED);      // (no region has number 0)
    return hipSuccess;
  }
  bool active() const { return words_ != nullptr; }
  CountPost where() const {
    if (!words_) return CountPost{nullptr, nullptr, 0};
    return CountPost{words_, n_ > n_counts_ ? words_ + n_counts_ : nullptr, r_.seq};
  }
  // Watches until every word is there and hands them to read(counts, channels).
  template <class Read>
  hipError_t wait(Read&& read) {
    uint32_t spins = 0;
    for (int64_t i = 0; i < n_;) {
      if (static_cast<uint32_t>(__atomic_load_n(words_ + i, __ATOMIC_ACQUIRE) >> 32) == r_.seq) { ++i; continue; }
#if defined(__x86_64__)
      __builtin_ia32_pause();
#endif
      if ((++spins & 0x3FFF) != 0) continue;
      const hipError_t e = hipStreamQuery(st_);       // (a failed launch or a fault ends the wait)
      if (e == hipErrorNotReady) continue;
      if (e == hipSuccess && static_cast<uint32_t>(__atomic_load_n(words_ + i, __ATOMIC_ACQUIRE) >> 32) == r_.seq) continue;
      return e != hipSuccess ? e : hipErrorUnknown;
    }
    read(static_cast<const uint64_t*>(words_), static_cast<const uint64_t*>(words_ + n_counts_));
    give_back();
    return hipSuccess;
  }

 private:
  void give_back() {
    r_.mark_done();
    g_staging[dev_].release(r_);
    if (r_.own) (void)hipHostFree(r_.own);
    words_ = nullptr;
  }
};

// Waits until everything queued on the stream is done, the caches' write-backs included: a launch that comes after it.
hipError_t stage_stream_idle(hipStream_t st) {
  StageRegion r;
  int dev = 0;
  const hipError_t e = stage_acquire(0, true, st, &r, &dev);
  if (e != hipSuccess) return e;
  CopyArgs a{};
  return stage_round_trip(a, dev, r, st, [] {});
}

// One table to the device; nothing waits (a table larger than half the ring aside).
hipError_t upload(void* dst, const void* src, size_t bytes, hipStream_t st) {
  if (bytes == 0) return hipSuccess;
  StageRegion r;
  int dev = 0;
  hipError_t e = stage_acquire(bytes, false, st, &r, &dev);
  if (e != hipSuccess) return e;
  std::memcpy(r.data, src, bytes);
  CopyArgs a{};
  a.add(r.data, dst, static_cast<int64_t>(bytes), kSrcHost);
  return stage_launch(a, r, true, st);
}

// Geometry of a ragged batch: one entry per item (sequence-major, head-minor).
struct Items {
  int64_t n_items = 0, total_tokens = 0;
  int32_t max_T = 0;
  std::vector<int32_t> T;          // [items]
  std::vector<int64_t> tok_off;    // [items]: first token of the item in ragged [hkv][T_s] arrays
  std::vector<int32_t> blk_off;    // [items]: first partition block
  int64_t n_blocks = 0;
};

Items make_items(const int32_t* seq_lens, int batch, int hkv) {
  Items it;
  int64_t off = 0;
  int64_t blk = 0;
  for (int s = 0; s < batch; ++s) {
    const int32_t T = seq_lens[s];
    it.max_T = std::max(it.max_T, T);
    for (int h = 0; h < hkv; ++h) {
      it.T.push_back(T);
      it.tok_off.push_back(off);
      it.blk_off.push_back(static_cast<int32_t>(blk));
      off += T;
      blk += (T + kPartBlock - 1) / kPartBlock;
    }
  }
  it.n_items = static_cast<int64_t>(batch) * hkv;
  it.total_tokens = off;
  it.n_blocks = blk;
  return it;
}

bool valid_tier(int b) { return b == 0 || b == 2 || b == 4 || b == 8 || b == 16; }

rdkv_status check_shape(int batch, int hq, int hkv, int d, const int32_t* seq_lens) {
  if (batch < 0 || hq <= 0 || hkv <= 0) return fail(RDKV_ERR_INVALID_ARG, "batch/hq/hkv must be positive");
  if (d != kHeadDim) return fail(RDKV_ERR_SHAPE, "head_dim %d unsupported (must be 128)", d);
  if (hq % hkv != 0) return fail(RDKV_ERR_SHAPE, "hq %d is not a multiple of hkv %d", hq, hkv);
  const int g = hq / hkv;
  if (!(g == 1 || g == 2 || g == 4 || g == 8)) return fail(RDKV_ERR_SHAPE, "hq/hkv = %d unsupported (1,2,4,8)", g);
  if (batch > 0 && seq_lens == nullptr) return fail(RDKV_ERR_INVALID_ARG, "seq_lens is null");
  int64_t total = 0;
  for (int s = 0; s < batch; ++s) {
    if (seq_lens[s] < 0) return fail(RDKV_ERR_SHAPE, "seq_lens[%d] = %d is negative", s, seq_lens[s]);
    total += static_cast<int64_t>(seq_lens[s]) * hkv;
  }
  if (total >= (1ll << 31)) return fail(RDKV_ERR_SHAPE, "sum of hkv*T_s exceeds 2^31 rows");
  return RDKV_OK;
}

rdkv_status check_config(const rdkv_config* cfg, bool need_budget, bool need_probe) {
  if (cfg == nullptr) return fail(RDKV_ERR_INVALID_ARG, "config is null");
  rdkv_status s = check_shape(cfg->batch, cfg->hq, cfg->hkv, cfg->head_dim, cfg->seq_lens);
  if (s != RDKV_OK) return s;
  if (cfg->group_size != kGroup && cfg->group_size != kHeadDim)
    return fail(RDKV_ERR_SHAPE, "group_size %d unsupported (32, or 128 = one scale per token row)", cfg->group_size);
  if (cfg->k_mode != RDKV_K_TOKENWISE && cfg->k_mode != RDKV_K_CHANNELWISE)
    return fail(RDKV_ERR_INVALID_ARG, "k_mode %d unknown", cfg->k_mode);
  if (need_probe) {
    if (cfg->s_obs <= 0 || cfg->s_obs > 64) return fail(RDKV_ERR_SHAPE, "s_obs %d out of range (1..64)", cfg->s_obs);
    if (cfg->pool_kernel < 1 || cfg->pool_kernel % 2 == 0 || cfg->pool_kernel > 15)
      return fail(RDKV_ERR_INVALID_ARG, "pool_kernel %d must be odd, 1..15", cfg->pool_kernel);
    for (int i = 0; i < cfg->batch; ++i)
      if (cfg->seq_lens[i] < cfg->s_obs)
        return fail(RDKV_ERR_SHAPE, "seq_lens[%d] = %d is shorter than s_obs = %d", i, cfg->seq_lens[i], cfg->s_obs);
  }
  if (need_budget) {
    if (cfg->batch > 0 && cfg->budget_bits == nullptr) return fail(RDKV_ERR_INVALID_ARG, "budget_bits is null");
    for (int i = 0; i < cfg->batch; ++i)
      if (!(cfg->budget_bits[i] >= 0.0f) || !std::isfinite(cfg->budget_bits[i]))
        return fail(RDKV_ERR_INVALID_ARG, "budget_bits[%d] must be finite and >= 0", i);
    if (cfg->n_tiers < 1 || cfg->n_tiers > RDKV_MAX_TIERS) return fail(RDKV_ERR_INVALID_ARG, "n_tiers out of range");
    for (int i = 0; i < cfg->n_tiers; ++i) {
      if (!valid_tier(cfg->tiers[i])) return fail(RDKV_ERR_INVALID_ARG, "tiers[%d] = %d not in {0,2,4,8,16}", i, cfg->tiers[i]);
      if (i > 0 && cfg->tiers[i] <= cfg->tiers[i - 1]) return fail(RDKV_ERR_INVALID_ARG, "tiers must be ascending");
      if (!std::isfinite(cfg->eps_v[i]) || !std::isfinite(cfg->eps_k[i]))
        return fail(RDKV_ERR_INVALID_ARG, "distortion table entry %d is not finite", i);
    }
    if (!(cfg->rel_tol >= 0.0f) || cfg->rel_tol >= 1.0f) return fail(RDKV_ERR_INVALID_ARG, "rel_tol must be in [0,1)");
    if (cfg->max_iters < 1 || cfg->max_iters > 200) return fail(RDKV_ERR_INVALID_ARG, "max_iters must be in 1..200");
    if (!(cfg->kv_split_rk > 0.0f) || !(cfg->kv_split_rk < 1.0f))
      return fail(RDKV_ERR_INVALID_ARG, "kv_split_rk must be in (0,1)");
  }
  return RDKV_OK;
}

// chunk size policy of the dense path; used by the workspace query and the launch alike.  The split kernel stages
// its tiles through 70 KB of LDS per workgroup, so a compute unit keeps two workgroups resident whatever the number
// of query heads: a launch is fastest when its workgroups fill the chip exactly once (512 chunks), and chunks have
// at least 256 rows.
void dense_plan(const int32_t* seq_lens, int batch, int hkv, int g, int* chunk_rows, int* max_splits) {
  int64_t total = 0;
  int max_T = 0;
  for (int s = 0; s < batch; ++s) {
    total += static_cast<int64_t>(seq_lens[s]) * hkv;
    max_T = std::max(max_T, seq_lens[s]);
  }
  (void)g;
  const int64_t resident = 512;
  int64_t cr = round_up(std::max<int64_t>(256, (total + resident - 1) / resident), 64);
  *chunk_rows = static_cast<int>(cr);
  *max_splits = std::max(1, static_cast<int>((max_T + cr - 1) / cr));
}

// Whether the launch merges its own partials (merge_tagged) instead of a second launch with a workgroup per query head.  The second
// launch takes the GPU 4.5 us and the host 3 (calls of less than 11.5 us are bound by the host with it, of 8.5 without).  One
// workgroup per item that reads all of its partials takes 2.7 us and 0.04 to 0.1 more for each of them: a win up to 48 of them
// (microseconds a call, two launches and one; chunks of an item x query heads per KV head):
//   2 items of 2K rows, 8 x 4      11.7   8.5      8 items of 8K, 32 x 1      11.8  10.7      128 items of 2K to 4K, 5 x 4   48.2  47.4
// and, over at most 16 MiB of rows, up to 64, at four heads 96:
//   8 items of 4K, 16 x 4          12.2   8.6      2 items of 6K, 24 x 4      12.4  10.8
// Beyond either, one compute unit's reading takes longer than the launch:
//   8 items of 8K, 32 x 4          11.8  13.8      32 items of 4K to 8K, 16 x 4  23.0  23.4   8 items of 32K, 64 x 4         29.3  32.7
// or does so where a graph replays the call and the host is out of it (2 items of 2K, 8 x 4: 8.8, 8.2; 2 of 6K, 24 x 4: 9.2, 9.2; 8 of
// 4K, 16 x 8: 10.6, 11.1; 2 of 12K, 47 x 2: 9.4, 9.5, 47 x 4: 9.8, 11.0).
constexpr int kDenseTagged = 64;       // chunks of an item that have room for their tags in its output rows, a lane each
static_assert(2 * kDenseTagged <= kHeadDim, "one query head's row");
bool dense_together(const int32_t* seq_lens, int batch, int hkv, int g, int max_splits) {
  const int partials = g * max_splits;
  if (max_splits > kDenseTagged || partials > (g == 4 ? 96 : 64)) return false;
  if (partials <= 48) return true;
  int64_t rows = 0;
  for (int s = 0; s < batch; ++s) rows += static_cast<int64_t>(seq_lens[s]) * hkv;
  return rows * (4 * kHeadDim) <= (static_cast<int64_t>(16) << 20);
}

// A tag that no other launch of the process has (DenseArgs::tag): two NaN patterns with 40 bits of a number between them, odd, so
// that they are no value of a bf16 number's bits either.
void next_tag(uint32_t (&tag)[2]) {
  static std::atomic<uint64_t> next{static_cast<uint64_t>(std::chrono::steady_clock::now().time_since_epoch().count()) * 0x9E3779B97F4A7C15ull};
  const uint64_t id = next.fetch_add(1, std::memory_order_relaxed);
  for (int i = 0; i < 2; ++i) tag[i] = 0xFFE00001u | (static_cast<uint32_t>(id >> (20 * i)) & 0xFFFFFu) << 1;
}

// What a cache owns on the device.  rdkv_pack takes one block for the arena and every table (one trip through the
// caller's allocator); what later calls add or replace (tail, rebuilt chunk tables, workspaces of other streams) are
// allocations of their own.
void free_cache_buffers(rdkv_cache* c) {
  Allocator al{c->alloc, c->free_, c->alloc_user};
  const uint8_t* b0 = c->d_block;
  const uint8_t* b1 = c->d_block ? c->d_block + c->block_bytes : nullptr;
  auto put = [&](void* p) {
    const uint8_t* q = static_cast<const uint8_t*>(p);
    if (p && !(b0 && q >= b0 && q < b1)) al.put(p);
  };
  put(c->d_arena);
  put(c->d_tier_idx);
  put(c->d_chunks);
  for (const rdkv_cache::Workspace& w : c->workspaces) put(w.block);
  c->workspaces.clear();
  put(c->d_tail_len);
  put(c->d_bits_tok);
  put(c->d_bits_ch);
  put(c->d_items_k);
  put(c->d_items_sched);
  put(c->d_tail);
  put(c->d_lambda);
  put(c->d_iters);
  al.put(c->d_block);
  c->d_block = nullptr;
  for (rdkv_cache* child : c->absorbed) {
    free_cache_buffers(child);
    delete child;
  }
  c->absorbed.clear();
}

// Memory of a split workspace for n_slots partials of a launch that looks for them or counts; the caller sets its first
// *absent bytes to merge::kAbsent, for a launch that looks, and the *arrive bytes at w->arrive to zero.
bool make_workspace(const rdkv_cache* c, hipStream_t st, int64_t n_slots, bool look, rdkv_cache::Workspace* w, size_t* absent,
                    size_t* arrive) {
  Allocator al{c->alloc, c->free_, c->alloc_user};
  const int g = c->hq / c->hkv;
  const size_t slots = static_cast<size_t>(std::max<int64_t>(n_slots, 1));
  const size_t acc_b = slots * g * (look ? merge::kRecordFloats : kHeadDim) * sizeof(float), ml_b = slots * g * 2 * sizeof(float);
  *absent = look ? acc_b : 0;
  *arrive = static_cast<size_t>(std::max<int64_t>(c->n_items, 1)) * sizeof(int32_t);
  uint8_t* block = static_cast<uint8_t*>(al.get(acc_b + ml_b + *arrive));
  if (!block) return false;
  *w = rdkv_cache::Workspace{st, reinterpret_cast<float*>(block), reinterpret_cast<float*>(block + acc_b),
                             reinterpret_cast<int32_t*>(block + acc_b + ml_b), block};
  return true;
}

// The split workspace of a cache for one stream (created on first use).  Calls on one stream are serialised by
// the stream and share a workspace; calls on different streams get different ones, so they may overlap.
rdkv_status workspace_for(const rdkv_cache* c, hipStream_t st, rdkv_cache::Workspace* out) {
  std::lock_guard<std::mutex> lk(c->ws_mu);
  for (const rdkv_cache::Workspace& w : c->workspaces)
    if (w.stream == st) { *out = w; return RDKV_OK; }
  // A stream under graph capture cannot allocate, and frameworks capture on streams of their own: a captured step
  // uses the cache's first workspace (the one of the stream that built the schedule).
  if (st != nullptr && !c->workspaces.empty()) {
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cs) == hipSuccess && cs == hipStreamCaptureStatusActive) {
      *out = c->workspaces.front();
      return RDKV_OK;
    }
  }
  rdkv_cache::Workspace w;
  size_t absent = 0, arrive = 0;
  if (!make_workspace(c, st, c->n_slots, c->merge_parts > 0, &w, &absent, &arrive)) return fail(RDKV_ERR_ALLOC, "device allocation of a split workspace failed");
  hipError_t e = hipMemsetAsync(w.arrive, 0, arrive, st);     // (the kernels keep both so)
  if (e == hipSuccess && absent > 0) e = hipMemsetAsync(w.block, 0xFF, absent, st);
  if (e != hipSuccess) {
    Allocator{c->alloc, c->free_, c->alloc_user}.put(w.block);
    return fail(RDKV_ERR_HIP, "clearing a split workspace: %s", hipGetErrorString(e));
  }
  c->workspaces.push_back(w);
  *out = w;
  return RDKV_OK;
}

void drop_workspaces(rdkv_cache* c) {
  std::lock_guard<std::mutex> lk(c->ws_mu);
  Allocator al{c->alloc, c->free_, c->alloc_user};
  for (const rdkv_cache::Workspace& w : c->workspaces) al.put(w.block);
  c->workspaces.clear();
}

// Launch order of a decode kernel's chunks.  Large launches: tier by tier, lowest bit-width first and largest first
// inside a tier, so that the chunks that cost most time per byte start first and the last to finish are 8-bit ones
// (measured 4-5 % faster on a mixed-tier batch than plain size order).  Launches that fit the chip in one round:
// round-robin over the items, so that with the usual round-robin placement of workgroups on the eight XCDs the
// chunks of an item share an L2 (which then also holds the partials their merge reads); only speed depends on it.
template <class T>      // Chunk or Piece
void order_chunks(typename std::vector<T>::iterator first, typename std::vector<T>::iterator last, int64_t n_items) {
  const int64_t count = last - first;
  if (count < 2) return;
  // (tier, size) in one key and the position behind it: a stable order without moving chunks about
  using Key = std::pair<uint64_t, int32_t>;
  auto key_of = [&](int64_t k) {
    const T& x = first[k];
    const uint64_t size = static_cast<uint64_t>(x.rows) * static_cast<uint64_t>(x.tier);
    return Key{(static_cast<uint64_t>(x.tier) << 48) + ((1ull << 48) - 1 - size), static_cast<int32_t>(k)};
  };
  std::vector<Key> key(count);
  std::vector<T> sorted;
  sorted.reserve(static_cast<size_t>(count));
  if (count > 1024 || n_items <= 1) {
    for (int64_t k = 0; k < count; ++k) key[k] = key_of(k);
    std::sort(key.begin(), key.end());
    for (int64_t k = 0; k < count; ++k) sorted.push_back(first[key[k].second]);
  } else {
    // each item's few chunks in that order, then dealt out a rank at a time (two sorts over all: 20 us more at 512)
    std::vector<int32_t> begin(static_cast<size_t>(n_items) + 1, 0);
    for (int64_t k = 0; k < count; ++k) ++begin[first[k].item + 1];
    for (int64_t i = 0; i < n_items; ++i) begin[i + 1] += begin[i];
    std::vector<int32_t> at(begin.begin(), begin.end() - 1);
    for (int64_t k = 0; k < count; ++k) key[at[first[k].item]++] = key_of(k);
    for (int64_t i = 0; i < n_items; ++i)
      if (!std::is_sorted(key.begin() + begin[i], key.begin() + begin[i + 1])) std::sort(key.begin() + begin[i], key.begin() + begin[i + 1]);
    for (int32_t rank = 0; static_cast<int64_t>(sorted.size()) < count; ++rank)
      for (int64_t i = 0; i < n_items; ++i)
        if (begin[i] + rank < begin[i + 1]) sorted.push_back(first[key[begin[i] + rank].second]);
  }
  std::copy(sorted.begin(), sorted.end(), first);
}

// Merging workgroups of an item in a launch that looks for its partials (8 g / parts blocks of 16 channels each, a wavefront
// each): four per query head while a launch has at most 128 of them; 0, the launch counts, where that takes more than 128
// or wavefronts with more than one block, i.e. from 129 query heads on (8 heads per KV head, four wavefronts a workgroup: 65).
// The places that chunks leave beside them (a compute unit holds one workgroup of these kernels, two with four wavefronts)
// are no line: 64 or 32 workgroups, or as many as there are places left, took 0 to 3 us more in launches of 175 to 241 chunks.
// Time looked for / time counted, caches cold, 4 to 1024 items of 300 to 20000 keys (lowest, geometric mean, highest; number of
// launches).  Token-wise launches of at most 256 chunks, 1 to 4 query heads per KV head:
//   up to 128 query heads  0.74 0.88 1.01  (148)     above  0.93 1.06 1.20  (26)
// 8 per KV head:
//   up to 64               0.82 0.93 1.05  (16)      above  0.95 1.19 1.46  (27)
// Channel-wise launches of eight-wavefront workgroups, whatever their number of chunks:
//   up to 128              0.84 0.94 1.06  (100)     above  0.97 1.03 1.11  (44)
int merge_parts(int g, int64_t n_items) {
  const int least = g > 4 ? 2 * g : g;
  if (least * n_items > 128) return 0;
  int parts = 4 * g;
  while (parts > least && parts * n_items > 128) parts /= 2;
  return parts;
}
// Their entries of the chunk table, written to where the table is put together (none for items whose only chunk writes the
// output rows itself).
int64_t count_merge_chunks(const std::vector<int32_t>& slot_count, int64_t n_items, int parts) {
  return parts * std::count_if(slot_count.begin(), slot_count.begin() + n_items, [](int32_t c) { return c > 1; });
}
void merge_chunks(const std::vector<int32_t>& slot_begin, const std::vector<int32_t>& slot_count, int64_t n_items, int parts, Chunk* to) {
  Chunk ch{};
  ch.tier = kTierMerge;
  ch.next = -1;
  for (int part = 0; part < parts; ++part)
    for (int64_t i = 0; i < n_items; ++i) {
      if (slot_count[i] <= 1) continue;
      ch.item = static_cast<int32_t>(i);
      ch.slot0 = slot_begin[i];
      ch.nslots = slot_count[i];
      ch.row0 = part;
      *to++ = ch;
    }
}

// A run of rows of one tier of one item while a schedule is put together.
struct Piece {
  int32_t item, tier;      // tier: bits
  int32_t row0, rows;
  int32_t slot, next;      // Chunk::slot, Chunk::next
};

// every chunk learns its item's first partial slot and slot count (the merge inside the decode kernels needs them)
void stamp_slots(std::vector<Chunk>& table, const std::vector<int32_t>& slot_begin, const std::vector<int32_t>& slot_count) {
  for (Chunk& ch : table) {
    ch.slot0 = slot_begin[ch.item];
    ch.nslots = slot_count[ch.item];
  }
}

// A channel map, eight channels at a time.
constexpr uint64_t kBytes01 = 0x0101010101010101ull;
uint64_t eight_channels(const uint8_t* bits_ch, int c) {
  uint64_t v;
  std::memcpy(&v, bits_ch + c, 8);
  return v;
}
bool valid_map(const uint8_t* bits_ch) {      // bits 1 to 4, one at most
  uint64_t bad = 0;
  for (int c = 0; c < kHeadDim; c += 8) {
    const uint64_t v = eight_channels(bits_ch, c);
    const uint64_t set = ((v >> 1) & kBytes01) + ((v >> 2) & kBytes01) + ((v >> 3) & kBytes01) + ((v >> 4) & kBytes01);
    bad |= (v & (kBytes01 * 0xE1)) | (set & (kBytes01 * 0xFE));
  }
  return bad == 0;
}
// Sorted-channel layout of one item's K tiles from its channel bit map.
// held: channels of every tier.  (A comparison per channel and tier, and a count of the slots that hold one, took 0.25 us an item, in
// front of the packing launch.)
ItemK make_item_k(const uint8_t* bits_ch, int32_t (&held)[4]) {
  ItemK k;
  std::memset(&k, 0, sizeof(k));
  std::memset(k.slot_ch, 0xFF, sizeof(k.slot_ch));      // -1
  int slot = 0, words = 0, qsteps = 0;
  for (int ti = 0; ti < 4; ++ti) {
    const int b = pack_tier_bits(ti);
    k.slot_base[ti] = static_cast<int16_t>(slot);
    int cnt = 0;
    for (int c = 0; c < kHeadDim; c += 8) {
      // bit i of the product's highest byte: channel c + i has the tier
      uint32_t has = static_cast<uint32_t>((((eight_channels(bits_ch, c) >> (4 - ti)) & kBytes01) * 0x0102040810204080ull) >> 56);
      for (; has != 0; has &= has - 1) k.slot_ch[slot + cnt++] = static_cast<int16_t>(c + __builtin_ctz(has));
    }
    held[ti] = cnt;
    const int npad = static_cast<int>(k_tier_slots(ti, static_cast<uint32_t>(cnt)));
    slot += npad;
    words += npad * b / 32;
    k.word_end[ti] = static_cast<int16_t>(words);
    if (ti == 0) k.n_steps16 = static_cast<int16_t>(npad / 4); else qsteps += npad / 4;
  }
  k.n_slots = static_cast<int16_t>(slot);
  k.n_qsteps = static_cast<int16_t>(qsteps);
  k.n_words = static_cast<int16_t>(words);
  k.n_words_padded = static_cast<int16_t>((words + 1) / 2 * 2);
  k.kt_bytes = k_tile_bytes(k.n_words_padded);
  k.km_bytes = k_meta_bytes(k.n_qsteps);
  return k;
}

// Lower convex hull of (b_k, eps_k) and the threshold ratios r_k = db / (-d eps) of its edges.
void hull_thresholds(const rdkv_config* cfg, const float* eps, std::vector<int>* tiers, std::vector<double>* r) {
  struct P { double b, e; };
  std::vector<P> h;
  for (int i = 0; i < cfg->n_tiers; ++i) {
    const P p{static_cast<double>(cfg->tiers[i]), static_cast<double>(eps[i])};
    while (h.size() >= 2) {
      const P& a = h[h.size() - 2];
      const P& b = h[h.size() - 1];
      const double cross = (b.b - a.b) * (p.e - a.e) - (b.e - a.e) * (p.b - a.b);
      if (cross <= 0.0) h.pop_back(); else break;
    }
    h.push_back(p);
  }
  tiers->clear();
  r->clear();
  tiers->push_back(static_cast<int>(h[0].b));
  for (size_t k = 1; k < h.size(); ++k) {
    const double de = h[k - 1].e - h[k].e;
    if (!(de > 0.0)) break;
    tiers->push_back(static_cast<int>(h[k].b));
    r->push_back((h[k].b - h[k - 1].b) / de);
  }
}


// What the kernels of one pass over a ragged batch read about it.  Up to kSeqsAlong sequences travel with the launches, a
// table of more goes to the device first.
struct Tables {
  Batch batch;
  int64_t n_tiles = 0;           // key tiles of all items
};

size_t table_bytes(int32_t n_seqs) { return n_seqs <= kSeqsAlong ? 0 : static_cast<size_t>(n_seqs) * sizeof(SeqEntry); }

rdkv_status make_tables(const rdkv_config* cfg, bool with_budget, Temp& tmp, hipStream_t st, Tables* out) {
  const bool mixed = cfg->k_mode == RDKV_K_CHANNELWISE;
  Batch& b = out->batch;
  std::memset(&b, 0, sizeof(b));
  b.n_seqs = cfg->batch;
  b.hkv = cfg->hkv;
  b.inv_hkv = cfg->hkv == 1 ? 0xFFFFFFFFu : static_cast<uint32_t>(((1ull << 32) + cfg->hkv - 1) / static_cast<uint64_t>(cfg->hkv));
  StageRegion region;
  int dev = 0;
  SeqEntry *entries = b.own, *d_table = nullptr;
  const size_t bytes = table_bytes(cfg->batch);
  if (bytes > 0) {
    d_table = tmp.get<SeqEntry>(static_cast<size_t>(cfg->batch));
    if (!d_table) return fail(RDKV_ERR_ALLOC, "device allocation failed");
    RDKV_HIP(stage_acquire(bytes, false, st, &region, &dev));
    entries = reinterpret_cast<SeqEntry*>(region.data);
  }
  int64_t row = 0, tile = 0, blk = 0;
  for (int s = 0; s < cfg->batch; ++s) {
    SeqEntry e{};
    e.row0 = row;
    e.T = cfg->seq_lens[s];
    e.tile0 = static_cast<int32_t>(tile);
    e.blk0 = static_cast<int32_t>(blk);
    if (with_budget) {
      // Stage 2.  Token-wise mode: the sequence's average serves K and V alike.  Channel-wise mode: V gets the share
      // 1 - r_K of the head budget, i.e. 2 (1 - r_K) avg_bits per token unit (rounded to fp32 like every budget).
      e.avg = cfg->budget_bits[s];
      e.budget = mixed ? static_cast<float>(2.0 * (1.0 - static_cast<double>(cfg->kv_split_rk)) * static_cast<double>(e.avg)) : e.avg;
    }
    entries[s] = e;
    const int64_t T = e.T;
    row += cfg->hkv * T;
    tile += cfg->hkv * ((T + kKeyTile - 1) / kKeyTile);
    blk += cfg->hkv * ((T + kPartBlock - 1) / kPartBlock);
  }
  out->n_tiles = tile;
  if (bytes > 0) {
    CopyArgs ca{};
    ca.add(region.data, d_table, static_cast<int64_t>(bytes), kSrcHost);
    RDKV_HIP(stage_launch(ca, region, true, st));
    b.table = d_table;
  }
  return RDKV_OK;
}

// Stage 1 of Alg. 1; everything is enqueued on st, nothing waits.  raw: see launch_weights.
rdkv_status weights_impl(const rdkv_config* cfg, const Items& it, const Tables& tb, const void* K, const void* Q_obs,
                         float* w_tok, float* w_ch, const float** raw, Temp& tmp, hipStream_t st) {
  const int R = cfg->hq / cfg->hkv * cfg->s_obs;
  const size_t nscr = weights_scratch_floats(tb.n_tiles, it.n_items, it.total_tokens, R, w_ch != nullptr);
  float* scratch = tmp.get<float>(nscr);
  if (!scratch) return fail(RDKV_ERR_ALLOC, "device allocation failed");
  TimedScope ts(RDKV_TIME_WEIGHTS, st);
  RDKV_HIP(launch_weights(*cfg, tb.batch, tb.n_tiles, it.n_items, it.total_tokens, it.max_T,
                          static_cast<const uint16_t*>(K), static_cast<const uint16_t*>(Q_obs), w_tok, w_ch, scratch,
                          raw, st));
  return RDKV_OK;
}

// Stages 2-3 of Alg. 1; everything is enqueued on st, nothing waits.  raw: weights that are still to be pooled into w_tok, or null.
// lam / iters: device [items] (token map), in channel-wise mode followed by [items] for the channel map; or null.
// blk_counts: device [blocks][4] for the packing stage (kept tokens of every block of an item per tier), or null.  post: see CountPost.
rdkv_status allocate_impl(const rdkv_config* cfg, const Items& it, const Tables& tb, const float* raw, float* w_tok,
                          const float* w_ch, uint8_t* bits_tok, uint8_t* bits_ch, double* lam, int32_t* iters,
                          int32_t* blk_counts, const CountPost& post, Temp& tmp, hipStream_t st) {
  const bool mixed = cfg->k_mode == RDKV_K_CHANNELWISE;
  const int n = static_cast<int>(it.n_items);
  std::vector<int> ht;
  std::vector<double> hr;
  hull_thresholds(cfg, cfg->eps_v, &ht, &hr);
  const size_t nscr = allocate_scratch_bytes(n, it.max_T);
  void* scratch = nscr ? tmp.get<uint8_t>(nscr) : nullptr;
  if (nscr && !scratch) return fail(RDKV_ERR_ALLOC, "device allocation failed");
  if (!blk_counts && mixed) {                 // Stage 3 starts from them
    blk_counts = tmp.get<int32_t>(static_cast<size_t>(std::max<int64_t>(it.n_blocks, 1)) * 4);
    if (!blk_counts) return fail(RDKV_ERR_ALLOC, "device allocation failed");
  }
  int32_t* d_order = nullptr;
  int n_long = 0, max_short = 0;
  if (allocate_needs_order(n, it.max_T)) {
    std::vector<int32_t> order(it.T.size());
    const auto is_long = [&](int32_t i) { return it.T[i] > allocate_short_units(); };
    for (int32_t i = 0; i < n; ++i)
      if (is_long(i)) order[n_long++] = i;
    for (int32_t i = 0, at = n_long; i < n; ++i)
      if (!is_long(i)) {
        order[at++] = i;
        max_short = std::max(max_short, it.T[i]);
      }
    d_order = tmp.get<int32_t>(order.size());
    if (!d_order) return fail(RDKV_ERR_ALLOC, "device allocation failed");
    RDKV_HIP(upload(d_order, order.data(), order.size() * sizeof(int32_t), st));
  }
  TimedScope ts(RDKV_TIME_ALLOCATE, st);      // every kernel of the stage
  RDKV_HIP(launch_allocate(raw, raw ? cfg->pool_kernel : 1, w_tok, tb.batch, it.max_T, d_order, n_long, max_short, static_cast<int>(ht.size()), ht.data(), hr.data(),
                           1.0 - static_cast<double>(cfg->rel_tol), cfg->max_iters, bits_tok, lam, iters,
                           blk_counts, post, scratch, st));
  if (!mixed) return RDKV_OK;
  // Stage 3, on the device: k_avg = min(16, 2 r_K avg_bits T / n_kept) over the retained tokens just counted
  hull_thresholds(cfg, cfg->eps_k, &ht, &hr);
  RDKV_HIP(launch_allocate_channels(w_ch, tb.batch, blk_counts, static_cast<double>(cfg->kv_split_rk),
                                    static_cast<int>(ht.size()), ht.data(), hr.data(),
                                    1.0 - static_cast<double>(cfg->rel_tol), cfg->max_iters, bits_ch,
                                    lam ? lam + n : nullptr, iters ? iters + n : nullptr, post, st));
  return RDKV_OK;
}

// d_blk_counts: the tier counts of every block of the bit map when the allocation has left them, or null; posted: what its kernels
// tell the host, or null; d_positions: scratch of a word per token when the caller has some, or null.
rdkv_status pack_impl(const rdkv_config* cfg, const Items& it, const Tables& tb, const void* K, const void* V,
                      const uint8_t* bits_tok, const uint8_t* bits_ch, int32_t* d_blk_counts, Posted* posted, int32_t* d_positions,
                      double* lam, int32_t* iters, Temp& tmp, hipStream_t st, rdkv_cache** out) {
  const bool mixed = cfg->k_mode == RDKV_K_CHANNELWISE;
  Allocator al{cfg->alloc, cfg->free_, cfg->alloc_user};
  const int g = cfg->hq / cfg->hkv;

  rdkv_cache* c = new (std::nothrow) rdkv_cache();
  if (!c) return fail(RDKV_ERR_ALLOC, "host allocation failed");
  c->batch = cfg->batch; c->hq = cfg->hq; c->hkv = cfg->hkv; c->d = cfg->head_dim; c->k_mode = cfg->k_mode;
  c->k_per_unit = (cfg->k_mode == RDKV_K_CHANNELWISE && cfg->k_scale_per_channel) ? 1 : 0;
  c->group_size = cfg->group_size;
  c->seq_lens.assign(cfg->seq_lens, cfg->seq_lens + cfg->batch);
  c->n_items = it.n_items; c->total_tokens = it.total_tokens;
  c->alloc = cfg->alloc; c->free_ = cfg->free_; c->alloc_user = cfg->alloc_user;
  auto bail = [&](rdkv_status code) { free_cache_buffers(c); delete c; return code; };
#define PACK_HIP(expr)                                                                             \
  do {                                                                                             \
    hipError_t e_ = (expr);                                                                        \
    if (e_ != hipSuccess) return bail(fail(RDKV_ERR_HIP, "%s: %s", #expr, hipGetErrorString(e_))); \
  } while (0)

  const int64_t n = it.n_items;
  c->counts.assign(n * 4, 0);
  c->seg_off.assign(n * 16, 0);
  const size_t n1 = static_cast<size_t>(std::max<int64_t>(n, 1));
  // tier counts of every block of the bit map: the allocation's own, or counted here
  const bool counted = d_blk_counts != nullptr;
  const int64_t n_counts = it.n_blocks * 4;
  if (!counted) d_blk_counts = tmp.get<int32_t>(n_counts);
  if (!d_positions) d_positions = tmp.get<int32_t>(it.total_tokens);
  PlanArgs plan{tmp.get<int64_t>(n1 * 4), tmp.get<int64_t>(n1 * 16), tmp.get<int32_t>(n1 * 4), mixed ? bits_ch : nullptr,
                mixed ? tmp.get<ItemK>(n1) : nullptr, static_cast<int32_t>(n), c->k_per_unit};
  // per-channel (minimum, maximum) over all retained tokens, as ordered integers
  uint32_t* d_krange = c->k_per_unit ? tmp.get<uint32_t>(n1 * kHeadDim * 2) : nullptr;
  if (!d_blk_counts || !d_positions || !plan.idx_base || !plan.seg_off || !plan.counts || (mixed && !plan.items_k) ||
      (c->k_per_unit && !d_krange))
    return bail(fail(RDKV_ERR_ALLOC, "device allocation failed"));
  std::vector<int32_t> k_bits(mixed ? n : 0), k_quantized(mixed ? n : 0);      // of an item's channels: bits, how many below 16
  if (n > 0) {
    // the one wait of the pass: the tier counts size the arena and the split schedule.  A kernel writes them into pinned
    // memory and the host watches for them (a copy to host memory and a wait for the stream: 25 us more).  It is the search's own
    // where that has posted them, and else the launch that makes the position lists and the packing kernels' tables, which need
    // nothing from here.
    if (!counted) {
      TimedScope ts(RDKV_TIME_PACK, st);      // first half of the stage: the tier counts
      PACK_HIP(launch_tier_count(bits_tok, tb.batch, d_blk_counts, it.max_T, st));
    }
    std::vector<uint8_t> h_bits_ch(mixed ? n * kHeadDim : 0);
    bool refused = false;
    if (posted && posted->active()) {
      // The allocation's kernels post their counts themselves: they are here when this launch starts on the device, and what the
      // host does next runs beside it (compressing 4K tokens 54.5 -> 52.7 us, 8 x 32K 111.0 -> 109.0).
      CopyArgs a{};
      if (d_krange) a.fill(d_krange, n * kHeadDim * 2 * static_cast<int64_t>(sizeof(uint32_t)), 0xFFFFFFFFu, 0u);
      plan_copy(a);
      {
        TimedScope ts(RDKV_TIME_PACK, st);
        PACK_HIP(launch_tier_scatter(bits_tok, tb.batch, d_blk_counts, d_positions, plan, it.max_T, a, st));
      }
      PACK_HIP(posted->wait([&](const uint64_t* counts, const uint64_t* channels) {
        for (int64_t i = 0; i < 4 * n; ++i) c->counts[i] = static_cast<int64_t>(counts[i] & 0xFFFFFFFFu);
        if (!mixed) return;
        for (int64_t i = 0; i < n; ++i)
          for (int w = 0; w < 16; ++w)
            for (uint32_t m = static_cast<uint32_t>(channels[16 * i + w]); m != 0; m &= m - 1)
              h_bits_ch[i * kHeadDim + 32 * (w & 3) + __builtin_ctz(m)] = static_cast<uint8_t>(16 >> (w >> 2));
      }));
    } else {
      const int64_t counts_b = round_up(n_counts * static_cast<int64_t>(sizeof(int32_t)), 16);
      StageRegion r;
      int dev = 0;
      PACK_HIP(stage_acquire(static_cast<size_t>(counts_b) + h_bits_ch.size(), true, st, &r, &dev));
      CopyArgs a{};
      a.add(d_blk_counts, r.data, n_counts * static_cast<int64_t>(sizeof(int32_t)), kDstHost);
      if (mixed) a.add(bits_ch, r.data + counts_b, static_cast<int64_t>(h_bits_ch.size()), kDstHost);
      if (d_krange) a.fill(d_krange, n * kHeadDim * 2 * static_cast<int64_t>(sizeof(uint32_t)), 0xFFFFFFFFu, 0u);
      const auto read = [&] {
        const int32_t* blk = reinterpret_cast<const int32_t*>(r.data);
        for (int64_t i = 0; i < n; ++i) {
          const int64_t b1 = i + 1 < n ? it.blk_off[i + 1] : it.n_blocks;
          int32_t sum[4] = {0, 0, 0, 0};
          for (int64_t b = it.blk_off[i]; b < b1; ++b) {
            refused = refused || blk[4 * b] < 0;      // (a block with a value that is no bit-width says so in its first count)
            for (int k = 0; k < 4; ++k) sum[k] += blk[4 * b + k];
          }
          for (int k = 0; k < 4; ++k) c->counts[i * 4 + k] = sum[k];
        }
        if (mixed) std::memcpy(h_bits_ch.data(), r.data + counts_b, h_bits_ch.size());
      };
      PACK_HIP(stage_round_trip(a, dev, r, st, read, [&](const CopyArgs& ca) {
        if (it.max_T == 0) return launch_copy(ca, st);      // no tokens, no lists
        TimedScope ts(RDKV_TIME_PACK, st);
        return launch_tier_scatter(bits_tok, tb.batch, d_blk_counts, d_positions, plan, it.max_T, ca, st);
      }));
    }
    if (refused) return bail(fail(RDKV_ERR_INVALID_ARG, "bits_tok holds a value outside {0, 2, 4, 8, 16}"));
    if (mixed) {
      c->items_k.resize(n);
      for (int64_t i = 0; i < n; ++i) {
        if (!valid_map(&h_bits_ch[i * kHeadDim])) {
          int ch = 0;
          while (ch < kHeadDim - 1 && valid_tier(h_bits_ch[i * kHeadDim + ch])) ++ch;
          return bail(fail(RDKV_ERR_INVALID_ARG, "bits_ch[%lld][%d] = %d is not a tier", static_cast<long long>(i),
                           ch, h_bits_ch[i * kHeadDim + ch]));
        }
        int32_t held[4];
        c->items_k[i] = make_item_k(&h_bits_ch[i * kHeadDim], held);
        for (int t2 = 0; t2 < 4; ++t2) {
          k_bits[i] += held[t2] * pack_tier_bits(t2);
          k_quantized[i] += t2 > 0 ? held[t2] : 0;
        }
        const ItemK& ik = c->items_k[i];
        if (ik.n_words_padded > kMaxKRowWords)
          return bail(fail(RDKV_ERR_INTERNAL, "K row of item %lld has %d words, more than the decode kernel holds (%d)",
                           static_cast<long long>(i), ik.n_words_padded, kMaxKRowWords));
        c->max_k_words = std::max<int32_t>(c->max_k_words, ik.n_words_padded);
        c->max_k_steps = std::max<int32_t>(c->max_k_steps, ik.n_steps16 + ik.n_qsteps);
        c->max_k_qsteps = std::max<int32_t>(c->max_k_qsteps, ik.n_qsteps);
      }
    }
  }

  // ---- plan: kept-position lists, arena segments, split schedule -------------------------
  int64_t kept = 0, cur = 0, stored = 0;
  int max_tiles = 0;
  for (int64_t i = 0; i < n; ++i) {
    int tiles = 0;
    const int64_t kbits = mixed ? k_bits[i] : 0, nquant = mixed ? k_quantized[i] : 0;      // of the item's channels
    for (int ti = 0; ti < 4; ++ti) {
      const int bits = pack_tier_bits(ti);
      const int64_t cnt = c->counts[i * 4 + ti];
      kept += cnt;
      tiles += static_cast<int>((cnt + kTile64 - 1) / kTile64);
      max_tiles = std::max(max_tiles, tiles);
      const SegmentUnits u = mixed ? segment_units(ti, static_cast<uint64_t>(cnt), true, c->items_k[i].n_words_padded, c->items_k[i].n_qsteps, c->k_per_unit)
                                   : segment_units(ti, static_cast<uint64_t>(cnt), false, 0, 0, false);
      const uint64_t sizes[4] = {u.k_data, u.k_meta, u.v_data, u.v_meta};
      for (int si = 0; si < 4; ++si) {
        c->seg_off[(i * 4 + ti) * 4 + si] = cur;
        cur += static_cast<int64_t>(sizes[si]) * kSegAlign;
      }
      if (mixed) {
        const int64_t groups = c->k_per_unit ? (cnt > 0 ? 1 : 0) : (cnt + kKTokenGroup - 1) / kKTokenGroup;
        stored += cnt * kbits / 8 + groups * 4 * nquant;
        stored += cnt * (tier_row_bytes(bits) + tier_meta_bytes(bits));
      } else {
        stored += cnt * 2 * (tier_row_bytes(bits) + tier_meta_bytes(bits));
      }
    }
  }
  c->arena_bytes = cur;
  c->kept_total = kept;
  c->stored_bytes = stored;

  // byte-balanced chunks: every workgroup streams about the same number of stored bytes.  Every chunk costs its
  // workgroup a hand-over at the end (partial stores that go through to memory and, in larger launches, an arrival atomic
  // whose answer the workgroup waits for) and its item one more partial to merge, so a launch wants exactly one round of workgroups:
  // as many chunks as the chip keeps resident (256 compute units x 2 workgroups of eight wavefronts = 512), never a
  // few more (measured on 4 x 128K tokens of 2-bit rows: 512 chunks 4.9 TB/s, 608 chunks 4.4, 2048 chunks 4.2).
  // Small launches are bound by latencies instead and are cut by rows (below); what is cut by bytes has chunks of at least
  // 96 KB.  Four-wavefront workgroups (8 query heads per KV head, channel-wise K) are cut into 768 chunks of at least 48 KB, three per
  // compute unit.  That is what the token-wise kernel keeps resident (157 registers).  Of the channel-wise ones, by their registers, a
  // compute unit has room for four with K rows of up to 16 words and one head set (126; and for two of eight wavefronts, where 256
  // in all are cut for), three up to 32 words (142), two with longer rows or two head sets (169 to 225); 768 was chosen when the first
  // of these had room for three, and other numbers have not been measured since.
  // channel-wise mode: eight-wavefront workgroups when the launch is small (one workgroup per compute unit holds
  // it) and the kernel has such an instantiation (up to 4 query heads per KV head, K rows of up to 32 words)
  const bool mixed_wide = mixed && g <= 4 && c->max_k_words <= 32 && stored < (static_cast<int64_t>(48) << 20);
  c->mixed_waves = mixed_wide ? 8 : 4;
  const bool wide = (!mixed && g <= 4) || mixed_wide;      // eight-wavefront workgroups
  const int64_t round_chunks = mixed_wide ? 256 : wide ? 512 : 768;
  // Cost of a row of a tier segment: its stored bytes, weighted in token-wise mode by what a byte of that tier costs
  // the decode kernel relative to an 8-bit byte (single-tier launches reach 4.92 / 5.41 / 5.68 / 5.38 TB/s on 2- /
  // 4- / 8- / 16-bit rows): in a launch of one round the slowest chunk sets the time, so chunks are balanced by
  // time, not bytes.
  auto row_cost = [&](int64_t i, int bits) -> int64_t {
    if (!mixed) {
      const int64_t pct = bits == 2 ? 115 : bits == 4 ? 105 : bits == 8 ? 100 : 106;
      return 2 * (tier_row_bytes(bits) + tier_meta_bytes(bits)) * pct / 100;
    }
    return tier_row_bytes(bits) + tier_meta_bytes(bits) + (c->items_k[i].kt_bytes + c->items_k[i].km_bytes + kTile64 - 1) / kTile64;
  };
  // (the 16-bit rows of a token-wise cache run in a kernel of their own and are cut separately below)
  const int ti0 = mixed ? 0 : 1;
  int64_t total_cost = 0, cost16 = 0;
  std::vector<int64_t> item_cost(n, 0);                       // of the tiers this launch cuts together
  for (int64_t i = 0; i < n; ++i) {
    for (int ti = ti0; ti < 4; ++ti) item_cost[i] += c->counts[i * 4 + ti] * row_cost(i, pack_tier_bits(ti));
    total_cost += item_cost[i];
    if (!mixed) cost16 += c->counts[i * 4] * row_cost(i, 16);
  }
  // Launches of up to kModelledCost are cut into rows, a multiple of 256 per chunk (one 64-row tile per SIMD), by a model of
  // their time: a start, the tiles that one SIMD goes through one after the other (8-bit rows take longer), and what each
  // chunk adds to the launch and each partial to the merge of its item.  A launch of at most 256 chunks has one workgroup per
  // compute unit and looks for its partials (or, with many query heads, counts: merge_parts); a larger one counts arrivals and
  // shares its compute units.  Against both stands the cut by bytes below, whose time goes with the bytes.  Fitted to 314
  // token-wise launches (2 to 64 items, 1 to 192 MB, up to 60 % 8-bit rows, caches cold).  244 others (1 to 128 items of even and
  // uneven lengths, 0.5 to 220 MB, 16-bit rows, tails) take 3.6 % less time in the geometric mean than with arrivals weighed as of a
  // counted merge and a line by bytes alone:
  // 55 of them at least 3 % less (one item of 220 MB, 8 heads per KV head: 717 chunks 62.7 us, 206 chunks 18.7), 8 more; 217 caches
  // of 0.4 to 8 bits per element and up to sixteen sequences 2.1 % less, 5 at least 3 % more (2 items of 23K rows: 62 chunks
  // 7.6 us, 184 chunks 8.0).
  // Some of the fit (microseconds per launch, number of chunks in parentheses):
  //   2 items, 8 MB                          k 1: 8.2 (236)   k 2: 7.4 (119)*  k 4: 8.6 (60)    by bytes: 8.3 (83)
  //   2 items, 64 MB                                          k 8: 16.8*       k 12: 19.9       by bytes: 22.9
  //   16 items, 64 MB, 60 % 8-bit rows                        k 6: 17.4*                        by bytes: 20.5
  //   16 items, 96 MB, 20 %                                   k 8: 26.9                         by bytes: 24.2*
  //   8 heads per KV head, 2 items, 64 MB, 60 %               k 4: 27.4 (280)  k 6: 21.5 (188)* by bytes: 42.9 (711)
  //   8 heads per KV head, 64 items, 64 MB                    k 4: 19.2 (477)*                  by bytes: 23.1 (1306)
  // Channel-wise launches of eight-wavefront workgroups (cut for one per compute unit, what rows of 17 to 32 words have room for) or
  // below the floor of the cut by bytes weigh their rounds, tiles and an item's partials instead (cut_channelwise).  Over 47
  // launches of one to sixteen sequences a model of the kind above was no faster (1.003) and up to 14 % slower (16 uneven
  // items of 8K to 24K rows), though 3 % faster over 216 even ones.
  constexpr double kModelledCost = 192e6;
  const int64_t floor_bytes = static_cast<int64_t>(wide ? 96 : 48) << 10;
  int64_t rows8 = 0, rows_all = 0;
  for (int64_t i = 0; i < n; ++i)
    for (int ti = ti0; ti < 4; ++ti) (ti == 1 ? rows8 : rows_all) += c->counts[i * 4 + ti];
  rows_all += rows8;
  const double share8 = static_cast<double>(rows8) / static_cast<double>(std::max<int64_t>(rows_all, 1));
  const double items = static_cast<double>(std::max<int64_t>(n, 1));
  // microseconds; tile8: more for each tile after the first free8 if all rows have 8 bits; byte: per 1e6 of cost
  struct LaunchTime { double start, tile, tile8, free8, chunk, partial, byte; };
  const LaunchTime alone = g > 4 ? LaunchTime{4.2, 1.6, 0.7, 2.0, 0.014, 0.0, 0.03} : LaunchTime{4.9, 0.25, 1.2, 3.0, 0.002, 0.001, 0.14};
  const LaunchTime among = g > 4 ? LaunchTime{4.4, 1.1, 0.67, 0.0, 0.008, 0.1, 0.0} : LaunchTime{1.7, 1.2, 0.69, 0.0, 0.018, 0.067, 0.0};
  struct Cut { int64_t rows; double time; };
  // Room for a tail's chunks, where they are few, so that the launch goes on looking: 8 items of 30K 4-bit rows in 240 chunks
  // 12.2 us, with a tail reserved 12.0.  (16 items of 8K in 256 chunks 9.5, with a tail's 16 more, counted, 11.7.)
  const int64_t room = n <= 8 ? 2 * n : 0;
  // the best rows per chunk for the tiers from ti_first on
  std::vector<uint32_t> segs;
  segs.reserve(static_cast<size_t>(n) * 4);
  auto cut_by_rows = [&](int ti_first, double share, bool only_looked) {
    constexpr uint32_t kMostTiles = 16;
    Cut best{0, 0.0};
    segs.clear();      // the 256 rows of each item and tier
    for (int64_t i = 0; i < n; ++i)
      for (int ti = ti_first; ti < 4; ++ti)
        if (c->counts[i * 4 + ti] > 0) segs.push_back((static_cast<uint32_t>(c->counts[i * 4 + ti]) + 255u) / 256u);
    for (uint32_t k = 1; k <= kMostTiles; k += g <= 4 && k >= 4 ? 2 : 1) {      // (eight wavefronts: 512 rows at a time)
      const uint32_t rows = 256u * k;
      int64_t n_wg = 0;
      uint32_t tiles = 0;      // of the largest chunk
      for (const uint32_t seg : segs) {
        const uint32_t nch = seg <= k ? 1u : (seg + k - 1) / k;
        n_wg += nch;
        if (tiles < std::min(seg, k)) tiles = std::max(tiles, (seg + nch - 1) / nch);
      }
      if (n_wg > 768 + 4 * n) continue;      // more than any launch needs, and than cache_max_table_bytes allows for
      const bool look = n_wg <= 256 - room;
      if (only_looked && !look) continue;
      const LaunchTime& t = look ? alone : among;
      const double rounds = static_cast<double>((n_wg + 255) / 256), depth = static_cast<double>(tiles);
      const double time = t.start + (t.tile * depth + t.tile8 * share * std::max(0.0, depth - t.free8)) * rounds +
                          (t.chunk + t.partial / items) * static_cast<double>(n_wg) + t.byte * 1e-6 * static_cast<double>(total_cost);
      if (best.rows == 0 || time < best.time) best = Cut{static_cast<int64_t>(rows), time};
    }
    return best;
  };
  const auto cut_channelwise = [&]() {
    Cut best{0, 0.0};
    for (uint32_t k = 1; k <= 16; k += k < 4 ? 1 : k < 8 ? 2 : 4) {
      const uint32_t rows = 256u * k;
      int64_t n_wg = 0, most = 0;
      for (int64_t i = 0; i < n; ++i) {
        int64_t slots = 0;
        for (int ti = 0; ti < 4; ++ti) slots += (static_cast<uint32_t>(c->counts[i * 4 + ti]) + rows - 1) / rows;
        n_wg += slots;
        most = std::max(most, slots);
      }
      if (n_wg > 768 + 4 * n && k < 16) continue;
      const double rounds = static_cast<double>((n_wg + round_chunks - 1) / round_chunks), at_once = static_cast<double>(most) / rounds;
      const double time = 6.5 * rounds + (g > 4 ? 6.0 : 3.0) * k * static_cast<double>((n_wg + 255) / 256) + 0.07 * at_once +
                          0.09 * std::max(0.0, at_once - 14.0);
      if (best.rows == 0 || time < best.time) best = Cut{static_cast<int64_t>(rows), time};
    }
    return best;
  };
  const auto by_bytes = [&](int64_t cost) { return std::min<int64_t>(round_chunks, cost / floor_bytes); };      // its chunks
  const auto bytes_time = [&](int64_t cost) {
    const double partials = static_cast<double>(by_bytes(cost)) / items;
    return g > 4 ? 10.0 + 0.16e-6 * static_cast<double>(cost) + 0.06 * partials : 8.1 + 0.118e-6 * static_cast<double>(cost) + 0.034 * partials;
  };
  int64_t small_rows = 0;
  if (mixed) {
    if (total_cost > 0 && (mixed_wide || total_cost <= round_chunks * floor_bytes)) small_rows = cut_channelwise().rows;
  } else if (total_cost > 0 && static_cast<double>(total_cost) <= kModelledCost) {
    const Cut cut = cut_by_rows(ti0, share8, false);
    if (by_bytes(total_cost) <= 256 || cut.time < bytes_time(total_cost)) small_rows = cut.rows;
  }
  // A token-wise launch of at most 256 chunks takes the 16-bit rows along (decode_tiles_take_rows): one launch instead of
  // two that follow each other (three short sequences of keep / 4 bit / evict 11.7 -> 8 us).  They take what 8-bit rows do.
  bool rows16_along = false;
  if (cost16 > 0 && total_cost + cost16 <= round_chunks * floor_bytes) {
    const Cut cut = cut_by_rows(0, 1.0, true);
    rows16_along = cut.rows > 0 && (total_cost + cost16 <= 256 * floor_bytes || cut.time < bytes_time(total_cost + cost16) + 4.0);
    if (rows16_along) small_rows = cut.rows;
  }
  // Number of chunks a chunk cost of cb gives, and the largest chunk's cost.  Chunks of less than an eighth of cb (a
  // tier with a handful of rows) do not count: they finish at once and leave their workgroup slot to the next chunk
  // (16 channel-wise sequences of 64K tokens, when the launch was half as fast: six even chunks per item and one tiny one, 899 in all
  // on 768 slots, took 108 us; five or seven per item 127-134 us).
  auto count_chunks = [&](int64_t cb, int64_t* max_cost) {
    int64_t total = 0;
    *max_cost = 0;
    for (int64_t i = 0; i < n; ++i)
      for (int ti = ti0; ti < 4; ++ti) {
        const int64_t cnt = c->counts[i * 4 + ti];
        if (cnt == 0) continue;
        const int64_t rc = row_cost(i, pack_tier_bits(ti));
        if (cnt * rc < cb / 8) continue;
        const int64_t want = std::max<int64_t>(64, cb / rc);
        const int64_t nch = (cnt + want - 1) / want;
        const int64_t rows_per = round_up((cnt + nch - 1) / nch, 64);
        total += (cnt + rows_per - 1) / rows_per;
        *max_cost = std::max(*max_cost, std::min(rows_per, cnt) * rc);
      }
    return total;
  };
  // token-wise mode cuts an item's quantized tiers as one run of work into round(cost / chunk cost) even shares
  auto count_shares = [&](int64_t cb, int64_t* max_cost) {
    int64_t total = 0;
    *max_cost = 0;
    for (int64_t i = 0; i < n; ++i)
      if (item_cost[i] > 0) total += std::max<int64_t>(1, (item_cost[i] + cb / 2) / cb);
    return total;
  };
  // Shares that span tiers pay a start-up per tier (operands rebuilt, the first tiles' latency waited for again):
  // worth it when a chunk streams for tens of microseconds (32 sequences x 128K tokens at 0.4 bit/elt: 101.6 -> 97.6
  // us), not in latency-bound launches (a 16 MB layer: 12.2 -> 13.7 us), which keep one tier per chunk.
  int64_t chunk_bytes = std::max<int64_t>(floor_bytes, total_cost / round_chunks);
  const bool shares = !mixed && small_rows == 0 && chunk_bytes >= (192 << 10);
  auto count_any = [&](int64_t cb, int64_t* max_cost) { return shares ? count_shares(cb, max_cost) : count_chunks(cb, max_cost); };
  int64_t max_cost = 0, n_one_round = count_any(chunk_bytes, &max_cost);
  for (int tries = 0; small_rows == 0 && tries < 64 && n_one_round > round_chunks + round_chunks / 50; ++tries) {   // (2 % over is fine)
    chunk_bytes += chunk_bytes / 16 + 1;
    n_one_round = count_any(chunk_bytes, &max_cost);
  }
  // When one round cannot be had (more tier segments than resident workgroups) or would be lopsided (its largest
  // chunk more than a fifth above the mean), about two rounds of smaller chunks even things out instead.
  // (Shares are even up to the rounding of an item's share count and stay in one round: 16 ragged sequences at 8
  // query heads per KV head, 728 chunks 52.9 us against 57.6 us for 1529.)
  if (small_rows == 0 && !shares && (n_one_round > round_chunks + round_chunks / 50 || max_cost * n_one_round > total_cost + total_cost / 5))
    chunk_bytes = std::max<int64_t>(floor_bytes, total_cost / (2 * round_chunks));
  // The row-major 16-bit kernel keeps two workgroups per compute unit resident (70 KB of LDS each): one round of
  // its own.
  const int64_t round16 = 512;
  const int64_t chunk_bytes16 = std::max<int64_t>(96 << 10, (cost16 + round16 - 1) / round16);
  std::vector<int32_t> slot_begin(std::max<int64_t>(n, 1), 0), slot_count(std::max<int64_t>(n, 1), 0);
  // (Cut and ordered as pieces, a quarter of a chunk's size, and written out once, into the memory the launch copies them from:
  // the packing launch waits for this.  728 chunks of 128 items took 25 us from the counts to the block's allocation; a pass
  // over them 645 -> 641 us, staged channel-wise calls on 50K keys 189 -> 185.)
  std::vector<Piece> pieces, conts;     // conts: continuation pieces (token-wise mode), reached through Chunk::next, never launched
  pieces.reserve(static_cast<size_t>(n_one_round + 2 * n));
  const auto make_piece = [](int64_t i, int ti, int64_t r0, int64_t rows) {
    return Piece{static_cast<int32_t>(i), pack_tier_bits(ti), static_cast<int32_t>(r0), static_cast<int32_t>(rows), 0, -1};
  };
  const auto chunk_of = [&](const Piece& p) {
    Chunk ch{};
    ch.tier = p.tier;
    ch.item = ch.reserved = p.item;
    ch.slot = p.slot;
    ch.next = p.next;
    ch.rows = p.rows;
    if (p.rows == 0) return ch;
    const int64_t i = p.item, r0 = p.row0;
    const int bits = p.tier, ti = bits == 16 ? 0 : bits == 8 ? 1 : bits == 4 ? 2 : 3;
    const int64_t* so = &c->seg_off[(i * 4 + ti) * 4];
    ch.k_data = so[0] + (mixed ? r0 / kTile64 * c->items_k[i].kt_bytes : r0 * tier_row_bytes(bits));
    ch.k_meta = so[1] + (mixed ? (c->k_per_unit ? 0 : r0 / kTile64 * c->items_k[i].km_bytes)
                               : r0 * tier_meta_bytes(bits));
    ch.v_data = so[2] + r0 * tier_row_bytes(bits);
    ch.v_meta = so[3] + r0 * tier_meta_bytes(bits);
    for (int t2 = 0; t2 < 4; ++t2) ch.k_word_end[t2] = mixed ? c->items_k[i].word_end[t2] : int16_t(0);
    return ch;
  };
  for (int64_t i = 0; i < n; ++i) {
    slot_begin[i] = static_cast<int32_t>(pieces.size());
    // segments cut tier by tier: every tier, or only the 16-bit tier (its own kernel) when the quantized tiers of a
    // token-wise item are cut into shares below
    for (int ti = 0; ti < (shares ? 1 : 4); ++ti) {
      const int bits = pack_tier_bits(ti);
      const int64_t cnt = c->counts[i * 4 + ti];
      if (cnt == 0) continue;
      const int64_t per_row = row_cost(i, bits);
      int64_t want = std::max<int64_t>(64, (!mixed && bits == 16 ? chunk_bytes16 : chunk_bytes) / per_row);
      if (small_rows > 0 && (mixed || bits != 16 || rows16_along)) want = small_rows;
      want = std::min<int64_t>(want, kMostChunkRows);
      const int64_t nch = (cnt + want - 1) / want;
      const int64_t rows_per = round_up((cnt + nch - 1) / nch, 64);
      for (int64_t r0 = 0; r0 < cnt; r0 += rows_per) {
        Piece p = make_piece(i, ti, r0, std::min<int64_t>(rows_per, cnt - r0));
        p.slot = static_cast<int32_t>(pieces.size());
        pieces.push_back(p);
      }
    }
    if (shares) {
      // The quantized tiers of a token-wise item are one run of work -- 2-bit rows, then 4-bit, then 8-bit -- cut
      // into equal shares of cost whatever the tiers' sizes: a workgroup's share may span two or three tiers (its
      // pieces are chained through Chunk::next and feed one softmax state), so every launch, single-tier or not,
      // gets chunks of even cost.
      const int64_t n_wg = item_cost[i] == 0 ? 0 : std::max<int64_t>(1, (item_cost[i] + chunk_bytes / 2) / chunk_bytes);
      int ti = 3;            // walk the segments from the 2-bit tier up
      int64_t r0 = 0;        // first row of the current segment not handed out yet
      for (int64_t k = 0; k < n_wg; ++k) {
        int64_t share = item_cost[i] / n_wg;     // what this workgroup should take
        int32_t prev = -1;                    // index of the workgroup's previous piece: >= 0 in conts, -2 - x: chunk x
        while (ti >= 1) {
          const int64_t left = c->counts[i * 4 + ti] - r0;
          if (left <= 0) { --ti; r0 = 0; continue; }
          const int64_t rc = row_cost(i, pack_tier_bits(ti));
          int64_t take = k + 1 == n_wg ? left : std::min<int64_t>(left, round_up(std::max<int64_t>(share, rc) / rc, 64));
          if (k + 1 < n_wg && left - take < 64) take = left;     // no slivers
          Piece p = make_piece(i, ti, r0, take);
          if (prev == -1) {
            p.slot = static_cast<int32_t>(pieces.size());
            pieces.push_back(p);
            prev = -2 - p.slot;
          } else {
            const int32_t me = static_cast<int32_t>(conts.size());
            conts.push_back(p);
            if (prev <= -2) pieces[-2 - prev].next = me; else conts[prev].next = me;   // local index for now
            prev = me;
          }
          r0 += take;
          share -= take * rc;
          if (k + 1 < n_wg && share < 64 * rc) break;            // the share is used up
        }
      }
    }
    if (static_cast<int32_t>(pieces.size()) == slot_begin[i]) {
      // nothing retained: an empty chunk, so that a workgroup still writes the item's output rows (0, lse = -inf)
      Piece p = make_piece(i, 3, 0, 0);
      p.slot = static_cast<int32_t>(pieces.size());
      pieces.push_back(p);
    }
    slot_count[i] = static_cast<int32_t>(pieces.size()) - slot_begin[i];
  }
  const int64_t n_launched = static_cast<int64_t>(pieces.size());
  c->n_slots = n_launched;
  // 16-bit chunks first (their own kernel), then the launched quantized ones, then the continuation pieces
  const int64_t n16 = std::count_if(pieces.begin(), pieces.end(), [](const Piece& x) { return x.tier == 16; });
  if (n16 > 0 && n16 < n_launched) std::stable_partition(pieces.begin(), pieces.end(), [](const Piece& x) { return x.tier == 16; });
  order_chunks<Piece>(pieces.begin(), pieces.begin() + n16, n);
  order_chunks<Piece>(pieces.begin() + n16, pieces.end(), n);
  c->n_chunks16 = n16;
  c->sched16 = n16;
  c->schedq = n_launched - n16;
  c->n_cont = static_cast<int64_t>(conts.size());
  // Chunk::next becomes an index into the whole table
  for (Piece& p : pieces) if (p.next >= 0) p.next += static_cast<int32_t>(n_launched);
  for (Piece& p : conts) if (p.next >= 0) p.next += static_cast<int32_t>(n_launched);
  // merging workgroups where the decode kernel looks for partials (see decode_merge.h)
  if (mixed ? c->mixed_waves == 8 : decode_tiles_take_rows(static_cast<int>(c->sched16 + c->schedq), c->n_cont > 0))
    c->merge_parts = merge_parts(g, n);
  c->n_merge = count_merge_chunks(slot_count, n, c->merge_parts);
  const int64_t n_chunks = n_launched + c->n_cont, n_table = n_chunks + c->n_merge;
  c->own_slot_count.assign(slot_count.begin(), slot_count.begin() + n);

  // ---- allocate what the cache owns: one block --------------------------------------------
  // [arena | appended tokens per item | arrival counters of this stream's workspace]  (cleared together)
  // [kept positions | token bit map | channel bit map | K row layouts, chunk table (one copy) | partials | lambda, steps]
  {
    auto up = [](int64_t b) { return round_up(std::max<int64_t>(b, 16), 256); };
    const int64_t o_state = c->arena_bytes, o_arrive = o_state + up(n * 4), o_idx = o_arrive + up(n * 4);
    const int64_t o_bt = o_idx + up(kept * 4), o_bc = o_bt + up(it.total_tokens);
    const int64_t o_ik = o_bc + (mixed ? up(n * kHeadDim) : 0);
    const int64_t ik_b = mixed ? round_up(n * static_cast<int64_t>(sizeof(ItemK)), 8) : 0;
    const int64_t o_acc = o_ik + up(ik_b + n_table * static_cast<int64_t>(sizeof(Chunk)));
    const int64_t o_ml = o_acc + up(std::max<int64_t>(c->n_slots, 1) * g * (c->merge_parts > 0 ? merge::kRecordFloats : kHeadDim) * 4);
    const int64_t o_lam = o_ml + up(std::max<int64_t>(c->n_slots, 1) * g * 2 * 4);
    const int maps = mixed ? 2 : 1;
    const int64_t o_it = o_lam + (lam ? up(maps * n * 8) : 0);
    const int64_t total = o_it + (iters ? up(maps * n * 4) : 0);
    c->d_block = static_cast<uint8_t*>(al.get(total));
    if (!c->d_block)
      return bail(fail(RDKV_ERR_ALLOC, "device allocation of the packed cache failed (%lld bytes)", static_cast<long long>(total)));
    c->block_bytes = total;
    c->d_arena = c->d_block;
    c->d_tail_len = reinterpret_cast<int32_t*>(c->d_block + o_state);
    c->d_tier_idx = reinterpret_cast<int32_t*>(c->d_block + o_idx);
    c->d_bits_tok = c->d_block + o_bt;
    if (mixed) {
      c->d_bits_ch = c->d_block + o_bc;
      c->d_items_k = reinterpret_cast<ItemK*>(c->d_block + o_ik);
    }
    c->d_chunks = reinterpret_cast<Chunk*>(c->d_block + o_ik + ik_b);
    c->index_bytes = total - c->arena_bytes;     // everything else in the block
    if (n > 0) {
      // the tables out of pinned memory, what the block keeps of the pass's scratch, the words that start at zero (the pack
      // kernels write every byte of the arena): in workgroups of the packing launch
      const int64_t tables_b = ik_b + n_table * static_cast<int64_t>(sizeof(Chunk));
      StageRegion r;
      int dev = 0;
      PACK_HIP(stage_acquire(static_cast<size_t>(tables_b), true, st, &r, &dev));
      if (mixed) std::memcpy(r.data, c->items_k.data(), n * sizeof(ItemK));
      // [launched chunks | continuation pieces | merging workgroups] (a schedule has one of the two last)
      Chunk* const table = reinterpret_cast<Chunk*>(r.data + ik_b);
      {
        Chunk* t = table;
        for (const Piece& p : pieces) {      // (they know their item's first partial slot and slot count)
          *t = chunk_of(p);
          t->slot0 = slot_begin[p.item];
          t->nslots = slot_count[p.item];
          ++t;
        }
        for (const Piece& p : conts) *t++ = chunk_of(p);
        merge_chunks(slot_begin, slot_count, n, c->merge_parts, t);
      }
      CopyArgs a{};
      a.add(r.data, c->d_block + o_ik, tables_b, kSrcHost);
      a.fill(c->d_block + o_state, o_idx - o_state, 0u, 0u);     // appended tokens, arrival counters
      if (c->merge_parts > 0) a.fill(c->d_block + o_acc, o_ml - o_acc, merge::kAbsent, merge::kAbsent);
      a.add(bits_tok, c->d_bits_tok, it.total_tokens);
      if (mixed) a.add(bits_ch, c->d_bits_ch, n * kHeadDim);
      if (lam) a.add(lam, c->d_block + o_lam, maps * n * 8);
      if (iters) a.add(iters, c->d_block + o_it, maps * n * 4);
      hipError_t launched = stage_launch(a, r, false, st, [&](const CopyArgs& ca) {
        if (kept == 0) return launch_copy(ca, st);
        TimedScope ts(RDKV_TIME_PACK, st);
        return launch_quant_pack(static_cast<const uint16_t*>(K), static_cast<const uint16_t*>(V), d_positions, c->d_tier_idx, plan,
                                 tb.batch, c->d_arena, max_tiles, d_krange, c->group_size == kHeadDim ? 1 : 0, ca, st);
      });
      if (launched == hipSuccess) c->chunks.assign(table, table + n_chunks);      // the host's copy, while the launch is on its way
      if (launched == hipSuccess && r.own) launched = stage_wait(r, st);
      g_staging[dev].release(r);
      if (r.own) (void)hipHostFree(r.own);
      PACK_HIP(launched);
      c->slot_begin = slot_begin;
      c->slot_count = slot_count;
      {   // the split workspace of this stream lives in the block: a first decode under graph capture allocates nothing
        std::lock_guard<std::mutex> lk(c->ws_mu);
        c->workspaces.push_back(rdkv_cache::Workspace{st, reinterpret_cast<float*>(c->d_block + o_acc),
                                                      reinterpret_cast<float*>(c->d_block + o_ml),
                                                      reinterpret_cast<int32_t*>(c->d_block + o_arrive), nullptr});
      }
    }
    if (lam) c->d_lambda = reinterpret_cast<double*>(c->d_block + o_lam);
    if (iters) c->d_iters = reinterpret_cast<int32_t*>(c->d_block + o_it);
  }

#undef PACK_HIP
  *out = c;
  return RDKV_OK;
}


}  // namespace

namespace rdkv {
void timing_begin(int kind, hipStream_t st) {
  std::lock_guard<std::mutex> lk(g_timing.mu);
  if (!g_timing.enabled) return;
  hipEvent_t a = g_timing.get(), b = g_timing.get();
  if (!a || !b) return;
  (void)hipEventRecord(a, st);
  g_timing.ev[kind].emplace_back(a, b);
}
void timing_end(int kind, hipStream_t st) {
  std::lock_guard<std::mutex> lk(g_timing.mu);
  if (!g_timing.enabled || g_timing.ev[kind].empty()) return;
  (void)hipEventRecord(g_timing.ev[kind].back().second, st);
}
}  // namespace rdkv

extern "C" {

rdkv_status rdkv_kernel_timing_enable(int32_t enable) {
  std::lock_guard<std::mutex> lk(g_timing.mu);
  g_timing.enabled = enable != 0;
  return RDKV_OK;
}

rdkv_status rdkv_kernel_timing_read(int32_t kind, int64_t* launches, double* total_ms) {
  if (kind < 0 || kind >= RDKV_TIME_KINDS || !launches || !total_ms)
    return fail(RDKV_ERR_INVALID_ARG, "bad timing kind or null output");
  std::lock_guard<std::mutex> lk(g_timing.mu);
  double sum = 0.0;
  int64_t n = 0;
  for (auto& pr : g_timing.ev[kind]) {
    float ms = 0.f;
    if (hipEventSynchronize(pr.second) == hipSuccess && hipEventElapsedTime(&ms, pr.first, pr.second) == hipSuccess) {
      sum += ms;
      ++n;
    }
    g_timing.pool.push_back(pr.first);
    g_timing.pool.push_back(pr.second);
  }
  g_timing.ev[kind].clear();
  *launches = n;
  *total_ms = sum;
  return RDKV_OK;
}

const char* rdkv_version(void) { return "rdkv-mi355x 0.1 (gfx950)"; }
const char* rdkv_last_error(void) { return g_err.c_str(); }

rdkv_status rdkv_config_default(rdkv_config* cfg) {
  if (!cfg) return fail(RDKV_ERR_INVALID_ARG, "config is null");
  std::memset(cfg, 0, sizeof(*cfg));
  cfg->head_dim = kHeadDim;
  cfg->s_obs = 32;
  cfg->pool_kernel = 5;
  cfg->causal = 1;
  cfg->k_mode = RDKV_K_TOKENWISE;
  cfg->group_size = kGroup;
  cfg->kv_split_rk = 0.5f;
  cfg->k_scale_per_channel = 0;
  cfg->n_tiers = 5;
  const int t[5] = {0, 2, 4, 8, 16};
  const float ev[5] = {1.0f, 0.313f, 0.0140f, 4.9e-5f, 0.0f};
  const float ek[5] = {1.0f, 0.149f, 0.0062f, 2.2e-5f, 0.0f};
  for (int i = 0; i < 5; ++i) {
    cfg->tiers[i] = t[i];
    cfg->eps_v[i] = ev[i];
    cfg->eps_k[i] = ek[i];
  }
  cfg->rel_tol = 1e-2f;
  cfg->max_iters = 64;
  return RDKV_OK;
}

rdkv_status rdkv_weights(const rdkv_config* cfg, const void* K, const void* Q_obs, float* w_tok,
                         float* w_ch, void* stream) {
  rdkv_status s = check_config(cfg, false, true);
  if (s != RDKV_OK) return s;
  if (cfg->batch == 0) return RDKV_OK;       // (the buffers of an empty batch may be null)
  if (!K || !Q_obs || !w_tok) return fail(RDKV_ERR_INVALID_ARG, "K, Q_obs and w_tok must not be null");
  hipStream_t st = static_cast<hipStream_t>(stream);
  Allocator al{cfg->alloc, cfg->free_, cfg->alloc_user};
  Temp tmp(al, st);
  Items it = make_items(cfg->seq_lens, cfg->batch, cfg->hkv);
  Tables tb;
  s = make_tables(cfg, false, tmp, st, &tb);
  if (s != RDKV_OK) return s;
  return weights_impl(cfg, it, tb, K, Q_obs, w_tok, w_ch, nullptr, tmp, st);
}

rdkv_status rdkv_calibrate_eps(const rdkv_config* cfg, const void* K, const void* V, double* eps_k, double* eps_v,
                               void* stream) {
  if (!cfg) return fail(RDKV_ERR_INVALID_ARG, "cfg must not be null");
  rdkv_status s = check_shape(cfg->batch, cfg->hq, cfg->hkv, cfg->head_dim, cfg->seq_lens);
  if (s != RDKV_OK) return s;
  if (cfg->k_mode != RDKV_K_TOKENWISE && cfg->k_mode != RDKV_K_CHANNELWISE)
    return fail(RDKV_ERR_INVALID_ARG, "k_mode must be RDKV_K_TOKENWISE or RDKV_K_CHANNELWISE");
  if (cfg->group_size != kGroup && cfg->group_size != kHeadDim)
    return fail(RDKV_ERR_SHAPE, "group_size %d unsupported (32, or 128 = one scale per token row)", cfg->group_size);
  if (!K || !V || !eps_k || !eps_v) return fail(RDKV_ERR_INVALID_ARG, "K, V, eps_k and eps_v must not be null");
  if (cfg->batch == 0) return RDKV_OK;
  for (int b = 0; b < cfg->batch; ++b)
    if (cfg->seq_lens[b] < 1) return fail(RDKV_ERR_SHAPE, "seq_lens[%d] = %d: calibration needs at least one token", b, cfg->seq_lens[b]);
  hipStream_t st = static_cast<hipStream_t>(stream);
  Allocator al{cfg->alloc, cfg->free_, cfg->alloc_user};
  s = refuse_capture(st);
  if (s != RDKV_OK) return s;
  Temp tmp(al, st);
  Items it = make_items(cfg->seq_lens, cfg->batch, cfg->hkv);
  const size_t n = static_cast<size_t>(it.n_items);
  const bool channelwise = cfg->k_mode == RDKV_K_CHANNELWISE;
  const bool whole = channelwise && cfg->k_scale_per_channel != 0;
  tmp.reserve({n * sizeof(int64_t), n * sizeof(int32_t), n * 8 * sizeof(double),
               whole ? n * kHeadDim * 2 * sizeof(uint32_t) : 0});
  int64_t* d_off = tmp.get<int64_t>(n);
  int32_t* d_T = tmp.get<int32_t>(n);
  double* d_acc = tmp.get<double>(n * 8);                       // [K | V][items][4]
  uint32_t* d_range = whole ? tmp.get<uint32_t>(n * kHeadDim * 2) : nullptr;
  if (!d_off || !d_T || !d_acc || (whole && !d_range)) return fail(RDKV_ERR_ALLOC, "device allocation failed");
  std::vector<double> h_acc(n * 8, 0.0);
  std::vector<uint32_t> h_range;
  RDKV_HIP(upload(d_off, it.tok_off.data(), n * sizeof(int64_t), st));
  RDKV_HIP(upload(d_T, it.T.data(), n * sizeof(int32_t), st));
  RDKV_HIP(upload(d_acc, h_acc.data(), h_acc.size() * sizeof(double), st));
  if (whole) {
    h_range.resize(n * kHeadDim * 2);
    for (size_t k = 0; k < h_range.size(); k += 2) { h_range[k] = 0xFFFFFFFFu; h_range[k + 1] = 0u; }
    RDKV_HIP(upload(d_range, h_range.data(), h_range.size() * sizeof(uint32_t), st));
  }
  {
    TimedScope ts(RDKV_TIME_CALIBRATE, st);
    RDKV_HIP(launch_calibrate(static_cast<const uint16_t*>(K), static_cast<const uint16_t*>(V), d_off, d_T,
                              static_cast<int>(n), it.max_T, channelwise, whole, cfg->group_size == kHeadDim, d_acc,
                              d_acc + n * 4, d_range, st));
  }
  RDKV_HIP(hipMemcpyAsync(h_acc.data(), d_acc, h_acc.size() * sizeof(double), hipMemcpyDeviceToHost, st));
  RDKV_HIP(hipStreamSynchronize(st));
  for (size_t i = 0; i < n; ++i)
    for (int side = 0; side < 2; ++side) {
      const double* a = h_acc.data() + (side * n + i) * 4;
      double* dst = (side == 0 ? eps_k : eps_v) + i * 3;
      for (int k = 0; k < 3; ++k) dst[k] = a[3] > 0.0 ? a[k] / a[3] : 0.0;
    }
  return RDKV_OK;
}

rdkv_status rdkv_allocate_info(const rdkv_config* cfg, const float* w_tok, const float* w_ch, uint8_t* bits_tok,
                               uint8_t* bits_ch, double* lambda_out, int32_t* iterations_out, void* stream) {
  rdkv_status s = check_config(cfg, true, false);
  if (s != RDKV_OK) return s;
  if (cfg->batch == 0) return RDKV_OK;       // (the buffers of an empty batch may be null)
  if (!w_tok || !bits_tok) return fail(RDKV_ERR_INVALID_ARG, "w_tok and bits_tok must not be null");
  const bool mixed = cfg->k_mode == RDKV_K_CHANNELWISE;
  if (mixed && (!w_ch || !bits_ch))
    return fail(RDKV_ERR_INVALID_ARG, "w_ch and bits_ch must not be null in channel-wise mode");
  hipStream_t st = static_cast<hipStream_t>(stream);
  Allocator al{cfg->alloc, cfg->free_, cfg->alloc_user};
  Temp tmp(al, st);
  Items it = make_items(cfg->seq_lens, cfg->batch, cfg->hkv);
  Tables tb;
  s = make_tables(cfg, true, tmp, st, &tb);
  if (s != RDKV_OK) return s;
  return allocate_impl(cfg, it, tb, nullptr, const_cast<float*>(w_tok), w_ch, bits_tok, bits_ch, lambda_out, iterations_out, nullptr, CountPost{},
                       tmp, st);
}

rdkv_status rdkv_allocate(const rdkv_config* cfg, const float* w_tok, const float* w_ch, uint8_t* bits_tok,
                          uint8_t* bits_ch, void* stream) {
  return rdkv_allocate_info(cfg, w_tok, w_ch, bits_tok, bits_ch, nullptr, nullptr, stream);
}

rdkv_status rdkv_pack(const rdkv_config* cfg, const void* K, const void* V, const uint8_t* bits_tok,
                      const uint8_t* bits_ch, void* stream, rdkv_cache** out) {
  if (out) *out = nullptr;
  rdkv_status s = check_config(cfg, false, false);
  if (s != RDKV_OK) return s;
  if (!out) return fail(RDKV_ERR_INVALID_ARG, "out is null");
  const bool mixed = cfg->k_mode == RDKV_K_CHANNELWISE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  Allocator al{cfg->alloc, cfg->free_, cfg->alloc_user};
  Items it = make_items(cfg->seq_lens, cfg->batch, cfg->hkv);
  if (it.total_tokens > 0 && (!K || !V || !bits_tok))
    return fail(RDKV_ERR_INVALID_ARG, "K, V and bits_tok must not be null");
  if (mixed && it.n_items > 0 && !bits_ch)
    return fail(RDKV_ERR_INVALID_ARG, "bits_ch must not be null in channel-wise mode");
  if (it.n_items > 0 && (s = refuse_capture(st)) != RDKV_OK) return s;
  Temp tmp(al, st);
  Tables tb;
  s = make_tables(cfg, false, tmp, st, &tb);
  if (s != RDKV_OK) return s;
  return pack_impl(cfg, it, tb, K, V, bits_tok, bits_ch, nullptr, nullptr, nullptr, nullptr, nullptr, tmp, st, out);
}

rdkv_status rdkv_compress(const rdkv_config* cfg, const void* K, const void* V, const void* Q_obs, void* stream,
                          rdkv_cache** out) {
  if (out) *out = nullptr;
  rdkv_status s = check_config(cfg, true, true);
  if (s != RDKV_OK) return s;
  if (!out) return fail(RDKV_ERR_INVALID_ARG, "out is null");
  const bool mixed = cfg->k_mode == RDKV_K_CHANNELWISE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  Allocator al{cfg->alloc, cfg->free_, cfg->alloc_user};
  Items it = make_items(cfg->seq_lens, cfg->batch, cfg->hkv);
  if (it.total_tokens > 0 && (!K || !V || !Q_obs)) return fail(RDKV_ERR_INVALID_ARG, "K, V and Q_obs must not be null");
  if (it.n_items > 0 && (s = refuse_capture(st)) != RDKV_OK) return s;
  Temp tmp(al, st);
  const size_t nt = static_cast<size_t>(std::max<int64_t>(it.total_tokens, 1));
  const size_t ni = static_cast<size_t>(std::max<int64_t>(it.n_items, 1));
  const size_t nc = ni * kHeadDim;
  {
    const int R = cfg->hq / cfg->hkv * cfg->s_obs;
    int64_t n_tiles = 0;
    for (int64_t i = 0; i < it.n_items; ++i) n_tiles += (it.T[i] + kKeyTile - 1) / kKeyTile;
    tmp.reserve({table_bytes(cfg->batch), nt * sizeof(float), nt, mixed ? nc * sizeof(float) : 0, mixed ? nc : 0,
                 weights_scratch_floats(n_tiles, it.n_items, it.total_tokens, R, mixed) * sizeof(float),
                 static_cast<size_t>(std::max<int64_t>(it.n_blocks * 4, 1)) * sizeof(int32_t), ni * 4 * sizeof(int64_t), ni * 16 * sizeof(int64_t),
                 ni * 4 * sizeof(int32_t), mixed ? ni * sizeof(ItemK) : 0, ni * 2 * sizeof(double), ni * 2 * sizeof(int32_t),
                 allocate_scratch_bytes(static_cast<int>(it.n_items), it.max_T),
                 allocate_needs_order(static_cast<int>(it.n_items), it.max_T) ? ni * sizeof(int32_t) : 0,
                 mixed && cfg->k_scale_per_channel ? nc * 2 * sizeof(uint32_t) : 0});
  }
  Tables tb;
  s = make_tables(cfg, true, tmp, st, &tb);
  if (s != RDKV_OK) return s;
  float* w = tmp.get<float>(nt);
  uint8_t* bits = tmp.get<uint8_t>(nt);
  float* w_ch = mixed ? tmp.get<float>(nc) : nullptr;
  uint8_t* bits_ch = mixed ? tmp.get<uint8_t>(nc) : nullptr;
  if (!w || !bits || (mixed && (!w_ch || !bits_ch))) return fail(RDKV_ERR_ALLOC, "device allocation failed");
  if (it.n_items == 0) return pack_impl(cfg, it, tb, K, V, bits, bits_ch, nullptr, nullptr, nullptr, nullptr, nullptr, tmp, st, out);
  // the multiplier and the step count of every item's search stay with the cache (rdkv_cache_stats / export): the
  // pack stage copies them into the cache's block
  const int maps = mixed ? 2 : 1;
  double* lam = tmp.get<double>(maps * ni);
  int32_t* iters = tmp.get<int32_t>(maps * ni);
  if (!lam || !iters) return fail(RDKV_ERR_ALLOC, "device allocation failed");
  const float* raw = nullptr;
  s = weights_impl(cfg, it, tb, K, Q_obs, w, w_ch, &raw, tmp, st);
  if (s != RDKV_OK) return s;
  int32_t* blk_counts = tmp.get<int32_t>(static_cast<size_t>(std::max<int64_t>(it.n_blocks, 1)) * 4);
  if (!blk_counts) return fail(RDKV_ERR_ALLOC, "device allocation failed");
  Posted posted;
  if (it.max_T > 0 && it.max_T <= allocate_short_units()) RDKV_HIP(posted.open(it.n_items, mixed, st));
  s = allocate_impl(cfg, it, tb, cfg->pool_kernel > 1 ? raw : nullptr, cfg->pool_kernel > 1 ? w : const_cast<float*>(raw), w_ch, bits, bits_ch, lam, iters, blk_counts,
                    posted.where(), tmp, st);
  if (s != RDKV_OK) return s;
  // (the weights are used up: their memory takes the kept positions)
  return pack_impl(cfg, it, tb, K, V, bits, bits_ch, blk_counts, &posted, reinterpret_cast<int32_t*>(w), lam, iters, tmp, st, out);
}

// A-priori bound on the packed arena from the budget alone (Sec. 3.2: sum of bit-widths <= floor(avg * units)).
// Token-wise: an item keeps at most B / b_min tokens (b_min = lowest stored bit-width of the tier set), and its rows
// cost 2 (16 b + 16) bytes each (no metadata at 16 bits), so at most 32 B + 32 B / b_min bytes, capped by all T rows
// at 16 bits; plus up to 63 padding rows per tier and the 256-byte alignment of its 16 segments.
// Channel-wise: V rows as above with the V share of the budget and one side only; a retained token's K row takes
// at most sum_c b_c / 8 <= 16 k_avg bytes of codes plus up to 24 bytes of segment padding, and a K tile of 64 tokens
// at most 32 bytes of metadata per quantized step (<= 35 steps).
static size_t cache_max_bytes(const rdkv_config* cfg) {
  const bool mixed = cfg->k_mode == RDKV_K_CHANNELWISE;
  int b_min = 16;
  for (int i = 0; i < cfg->n_tiers; ++i)
    if (cfg->tiers[i] > 0) b_min = std::min(b_min, cfg->tiers[i]);
  double total = 0.0;
  for (int s = 0; s < cfg->batch; ++s) {
    const double T = static_cast<double>(cfg->seq_lens[s]);
    const double a = static_cast<double>(cfg->budget_bits[s]);
    double item;
    if (!mixed) {
      const double B = std::min(std::floor(a * T), 16.0 * T);
      const double kept = std::min(B / b_min, T);
      item = std::min(32.0 * B + 32.0 * kept, 512.0 * T) + 63.0 * 2.0 * (256 + 144 + 80 + 48);
    } else {
      const double rk = static_cast<double>(cfg->kv_split_rk);
      const double Bv = std::min(std::floor(static_cast<double>(static_cast<float>(2.0 * (1.0 - rk) * a)) * T), 16.0 * T);
      const double kept = std::min(Bv / b_min, T);
      const double v = std::min(16.0 * Bv + 16.0 * kept, 256.0 * T) + 63.0 * (256 + 144 + 80 + 48);
      // K: codes <= 16 * (2 r_K a T) bytes over all kept tokens (k_avg n_kept = 2 r_K a T), at most 256 per token
      const double k_codes = std::min(16.0 * 2.0 * rk * a * T, 256.0 * kept) + 24.0 * kept;
      const double tiles = std::ceil(kept / 64.0) + 4.0;
      item = v + k_codes + tiles * 32.0 * 35.0 + 4.0 * 63.0 * 4.0 * kMaxKRowWords;
    }
    total += cfg->hkv * (item + 16.0 * kSegAlign);
  }
  return static_cast<size_t>(total) + kSegAlign;
}

// The same for everything else in the cache's block: kept positions (4 bytes each), the bit maps, the K row layouts,
// the chunk table and the first split workspace (at most two rounds of chunks and eight per item, g x 258 floats each, and
// the merging workgroups), lambda and step counts, and the alignment of the parts.
static size_t cache_max_table_bytes(const rdkv_config* cfg) {
  const bool mixed = cfg->k_mode == RDKV_K_CHANNELWISE;
  const int g = cfg->hq / cfg->hkv;
  int b_min = 16;
  for (int i = 0; i < cfg->n_tiers; ++i)
    if (cfg->tiers[i] > 0) b_min = std::min(b_min, cfg->tiers[i]);
  double kept = 0.0, tokens = 0.0;
  for (int s = 0; s < cfg->batch; ++s) {
    const double T = static_cast<double>(cfg->seq_lens[s]);
    const double a = static_cast<double>(cfg->budget_bits[s]) * (mixed ? 2.0 * (1.0 - static_cast<double>(cfg->kv_split_rk)) : 1.0);
    kept += cfg->hkv * std::min(std::floor(a * T) / b_min, T);
    tokens += cfg->hkv * T;
  }
  const double items = static_cast<double>(cfg->batch) * cfg->hkv;
  const double chunks = 2.0 * 768.0 + 8.0 * items;
  return static_cast<size_t>(4.0 * kept + tokens + items * (kHeadDim + sizeof(ItemK) + 8 + 2 * 12) +
                             chunks * (sizeof(Chunk) + g * (merge::kRecordFloats + 2) * 4.0) + 128.0 * sizeof(Chunk) +
                             16.0 * 256);
}

size_t rdkv_cache_max_bytes(const rdkv_config* cfg) {
  if (check_config(cfg, true, false) != RDKV_OK) return 0;
  return cache_max_bytes(cfg);
}

size_t rdkv_cache_max_table_bytes(const rdkv_config* cfg) {
  if (check_config(cfg, true, false) != RDKV_OK) return 0;
  return cache_max_table_bytes(cfg);
}

// Wavefronts per workgroup of a channel-wise schedule whose longest K row over all generations has sched_k_words words
// (0: there is one generation).
static int sched_mixed_waves(const rdkv_cache* c, int32_t sched_k_words) {
  return std::max(c->max_k_words, sched_k_words) <= 32 && c->hq / c->hkv <= 4 ? c->mixed_waves : 4;
}
// Some workgroup of a token-wise schedule goes through more than one tier of its item.
static bool sched_multi(const rdkv_cache* c) {
  bool multi = c->n_cont > 0;
  for (const rdkv_cache* child : c->absorbed) multi = multi || child->n_cont > 0;
  return multi;
}

rdkv_status rdkv_decode_attn(const rdkv_cache* c, const void* q, float* out, float* lse, void* stream) {
  if (!c) return fail(RDKV_ERR_INVALID_ARG, "cache must not be null");
  if (c->n_items == 0) return RDKV_OK;       // nothing to compute (and q / out of an empty batch may be null)
  if (!q || !out) return fail(RDKV_ERR_INVALID_ARG, "q and out must not be null");
  hipStream_t st = static_cast<hipStream_t>(stream);
  rdkv_cache::Workspace w;
  const rdkv_status ws = workspace_for(c, st, &w);
  if (ws != RDKV_OK) return ws;
  const int g = c->hq / c->hkv;
  const MergeArgs ma{w.part_acc, w.part_ml, w.arrive, out, lse, g, c->merge_parts, c->looks};
  // every chunk of the schedule is launched, the tail's included: chunks of tail rows that do not exist yet find
  // the current length in the cache's device word and contribute an empty partial
  const int n16 = static_cast<int>(c->sched16), nrest = static_cast<int>(c->schedq + c->n_tail_chunks);
  const int n_merge = static_cast<int>(c->n_merge);
  TimedScope ts(RDKV_TIME_DECODE_TIERED, st);
  if (c->k_mode == RDKV_K_CHANNELWISE) {
    RDKV_HIP(launch_decode_mixed(c->d_chunks, n16 + nrest + n_merge, c->d_arena, c->d_items_sched ? c->d_items_sched : c->d_items_k,
                                 std::max(c->max_k_words, c->sched_k_words), std::max(c->max_k_steps, c->sched_k_steps),
                                 std::max(c->max_k_qsteps, c->sched_k_qsteps), static_cast<const uint16_t*>(q), ma,
                                 c->d_tail_len, c->k_per_unit, sched_mixed_waves(c, c->sched_k_words), st));
    return RDKV_OK;
  }
  const bool multi = sched_multi(c);
  const uint16_t* qp = static_cast<const uint16_t*>(q);
  if (decode_tiles_take_rows(n16 + nrest, multi)) {     // one launch for all tiers
    RDKV_HIP(launch_decode_tiles(c->d_chunks, 0, n16 + nrest, n_merge, n16 > 0, multi, c->d_arena, qp, ma, c->d_tail_len, st));
    return RDKV_OK;
  }
  // the workgroups of both kernels announce themselves on the same counters: whichever finishes an item merges it
  RDKV_HIP(launch_decode_tiered_split(c->d_chunks, n16, c->d_arena, qp, ma, st));
  RDKV_HIP(launch_decode_tiles(c->d_chunks, n16, nrest, 0, false, multi, c->d_arena, qp, ma, c->d_tail_len, st));
  return RDKV_OK;
}

// Rebuilds the decode schedule of a cache: the chunks of the cache itself and of every absorbed generation (all
// 16-bit chunks first, then the quantized ones), then the tail's chunks in (chunk index, item) order so that the
// live ones are a prefix.  Every item keeps its partial slots contiguous: own chunks, generation by generation,
// then the tail.  The decode kernels address everything relative to d_arena, so the offsets of the other
// allocations are pointer differences.  `clear`: memory of the caller's that the same launch clears.  Waits for the stream;
// on failure the cache is unchanged.
static rdkv_status rebuild_schedule(rdkv_cache* c, void* clear, int64_t clear_bytes, hipStream_t st) {
  Allocator al{c->alloc, c->free_, c->alloc_user};
  const int64_t n = c->n_items;
  const int npi = (c->tail_cap + kTailChunkRows - 1) / kTailChunkRows;     // tail chunks per item
  std::vector<const rdkv_cache*> gens{c};
  gens.insert(gens.end(), c->absorbed.begin(), c->absorbed.end());
  std::vector<int32_t> nb(n), nc(n);
  std::vector<std::vector<int32_t>> gen_off(gens.size(), std::vector<int32_t>(n));
  int64_t n_slots = 0, n_gen_chunks = 0;
  for (int64_t i = 0; i < n; ++i) {
    nb[i] = static_cast<int32_t>(n_slots);
    int32_t off = 0;
    for (size_t k = 0; k < gens.size(); ++k) {
      gen_off[k][i] = off;
      off += gens[k]->own_slot_count[i];
    }
    nc[i] = off + npi;
    n_slots += nc[i];
  }
  // table = [16-bit chunks of every generation | launched quantized chunks of every generation | tail chunks |
  //          merging workgroups | continuation pieces of every generation];
  // a generation's own vector is [16-bit | launched | continuations]
  int64_t n_cont_total = 0;
  std::vector<int64_t> cont_off(gens.size());
  for (size_t k = 0; k < gens.size(); ++k) {
    n_gen_chunks += static_cast<int64_t>(gens[k]->chunks.size()) - gens[k]->n_cont;
    cont_off[k] = n_cont_total;
    n_cont_total += gens[k]->n_cont;
  }
  // channel-wise K: every (generation, item) has its own sorted-channel row layout
  const bool mixed = c->k_mode == RDKV_K_CHANNELWISE;
  std::vector<ItemK> items_sched;
  int32_t kw = 0, ks = 0, kq = 0;
  if (mixed && gens.size() > 1) {
    for (const rdkv_cache* gc : gens) {
      items_sched.insert(items_sched.end(), gc->items_k.begin(), gc->items_k.end());
      kw = std::max(kw, gc->max_k_words);
      ks = std::max(ks, gc->max_k_steps);
      kq = std::max(kq, gc->max_k_qsteps);
    }
  }
  int parts = 0;      // where the decode kernel looks for partials
  if (mixed ? sched_mixed_waves(c, kw) == 8 : decode_tiles_take_rows(static_cast<int>(n_gen_chunks + n * npi), sched_multi(c)))
    parts = merge_parts(c->hq / c->hkv, n);
  const int64_t n_merge = count_merge_chunks(nc, n, parts);
  const int64_t cont_base = n_gen_chunks + n * npi + n_merge;      // where the continuation pieces start in the new table
  std::vector<Chunk> table;
  table.reserve(static_cast<size_t>(cont_base + n_cont_total));
  std::vector<Chunk> own = c->chunks;   // this cache's chunks with their new slot numbers
  int64_t n16 = 0;
  auto moved = [&](size_t k, Chunk ch) {
    const rdkv_cache* gc = gens[k];
    const int64_t base = reinterpret_cast<intptr_t>(gc->d_arena) - reinterpret_cast<intptr_t>(c->d_arena);
    ch.reserved = static_cast<int32_t>(k * n + ch.item);
    ch.k_data += base;
    ch.k_meta += base;
    ch.v_data += base;
    ch.v_meta += base;
    if (ch.next >= 0) {   // an index into the generation's own vector -> into the new table
      const int64_t first_cont = static_cast<int64_t>(gc->chunks.size()) - gc->n_cont;
      ch.next = static_cast<int32_t>(cont_base + cont_off[k] + (ch.next - first_cont));
    }
    return ch;
  };
  for (int pass = 0; pass < 2; ++pass)
    for (size_t k = 0; k < gens.size(); ++k) {
      const rdkv_cache* gc = gens[k];
      const size_t launched = gc->chunks.size() - static_cast<size_t>(gc->n_cont);
      for (size_t j = 0; j < launched; ++j) {
        Chunk ch = gc->chunks[j];
        if ((ch.tier == 16) != (pass == 0)) continue;
        ch.slot = nb[ch.item] + gen_off[k][ch.item] + (ch.slot - gc->slot_begin[ch.item]);
        if (k == 0) own[j].slot = ch.slot;
        table.push_back(moved(k, ch));
        n16 += pass == 0;
      }
    }
  const int64_t tail_tiles = (c->tail_cap + kTile64 - 1) / kTile64, tile_bytes = kTile64 * kHeadDim * 2;
  const int64_t side = n * tail_tiles * tile_bytes;     // K tiles of all items, then V tiles
  const int64_t tail_base = reinterpret_cast<intptr_t>(c->d_tail) - reinterpret_cast<intptr_t>(c->d_arena);
  for (int j = 0; j < npi; ++j)
    for (int64_t i = 0; i < n; ++i) {
      Chunk ch;
      std::memset(&ch, 0, sizeof(ch));
      ch.k_data = tail_base + (i * tail_tiles + static_cast<int64_t>(j) * (kTailChunkRows / kTile64)) * tile_bytes;
      ch.v_data = ch.k_data + side;
      ch.rows = std::min<int32_t>(kTailChunkRows, c->tail_cap - j * kTailChunkRows);
      ch.tier = kTierTail;
      ch.item = static_cast<int32_t>(i);
      ch.slot = nb[i] + nc[i] - npi + j;
      ch.row0 = j * kTailChunkRows;
      ch.next = -1;
      table.push_back(ch);
    }
  table.resize(table.size() + static_cast<size_t>(n_merge));
  merge_chunks(nb, nc, n, parts, table.data() + (table.size() - static_cast<size_t>(n_merge)));
  for (size_t k = 0; k < gens.size(); ++k) {
    const rdkv_cache* gc = gens[k];
    for (size_t j = gc->chunks.size() - static_cast<size_t>(gc->n_cont); j < gc->chunks.size(); ++j)
      table.push_back(moved(k, gc->chunks[j]));
  }
  // launch order inside each kernel's range; the tail's chunks and the continuation pieces stay where they are
  order_chunks<Chunk>(table.begin(), table.begin() + n16, n);
  order_chunks<Chunk>(table.begin() + n16, table.begin() + n_gen_chunks, n);
  stamp_slots(table, nb, nc);
  stamp_slots(own, nb, nc);
  const int64_t n_table = static_cast<int64_t>(table.size());
  ItemK* d_items_sched = nullptr;
  if (!items_sched.empty()) {
    d_items_sched = static_cast<ItemK*>(al.get(items_sched.size() * sizeof(ItemK)));
    if (!d_items_sched) return fail(RDKV_ERR_ALLOC, "device allocation failed");
  }
  Chunk* d_chunks = static_cast<Chunk*>(al.get(std::max<int64_t>(n_table, 1) * sizeof(Chunk)));
  if (!d_chunks) {
    al.put(d_items_sched);
    return fail(RDKV_ERR_ALLOC, "device allocation failed");
  }
  rdkv_cache::Workspace w;   // this stream's workspace right away: a decode under graph capture then allocates nothing
  size_t absent = 0, arrive = 0;
  const bool have_w = make_workspace(c, st, n_slots, parts > 0, &w, &absent, &arrive);   // (a failure is reported by the decode call that needs it)
  // tables up, the workspace and the caller's memory set in one launch; the stream must be idle before the old tables and
  // workspaces go: a decode step may still be reading them
  const size_t table_b = table.size() * sizeof(Chunk), items_b = items_sched.size() * sizeof(ItemK);
  StageRegion r;
  int dev = 0;
  hipError_t e = stage_acquire(table_b + items_b, false, st, &r, &dev);
  if (e == hipSuccess) {
    if (table_b > 0) std::memcpy(r.data, table.data(), table_b);
    if (items_b > 0) std::memcpy(r.data + table_b, items_sched.data(), items_b);
    CopyArgs a{};
    a.add(r.data, d_chunks, static_cast<int64_t>(table_b), kSrcHost);
    a.add(r.data + table_b, d_items_sched, static_cast<int64_t>(items_b), kSrcHost);
    a.fill(clear, clear_bytes, 0u, 0u);
    if (have_w) a.fill(w.arrive, static_cast<int64_t>(arrive), 0u, 0u);
    if (have_w) a.fill(w.block, static_cast<int64_t>(absent), merge::kAbsent, merge::kAbsent);
    e = stage_launch(a, r, true, st);
  }
  if (e == hipSuccess) e = stage_stream_idle(st);
  if (e != hipSuccess) {
    al.put(d_chunks); al.put(d_items_sched);
    if (have_w) al.put(w.block);
    return fail(RDKV_ERR_HIP, "rebuilding the decode schedule: %s", hipGetErrorString(e));
  }
  drop_workspaces(c);      // the slot count changed: workspaces are created again on first use
  c->n_slots = n_slots;
  {   // the first chunk table lives in the cache's block; rebuilt ones are allocations of their own
    const uint8_t* q = reinterpret_cast<const uint8_t*>(c->d_chunks);
    if (!(c->d_block && q >= c->d_block && q < c->d_block + c->block_bytes)) al.put(c->d_chunks);
  }
  al.put(c->d_items_sched);
  c->d_items_sched = d_items_sched;
  c->sched_k_words = kw;
  c->sched_k_steps = ks;
  c->sched_k_qsteps = kq;
  c->d_chunks = d_chunks;
  c->sched16 = n16;
  c->schedq = n_gen_chunks - n16;
  c->n_tail_chunks = n * npi;
  c->n_merge = n_merge;
  c->merge_parts = parts;
  c->chunks.swap(own);
  c->slot_begin.swap(nb);
  c->slot_count.swap(nc);
  if (have_w) {
    std::lock_guard<std::mutex> lk(c->ws_mu);
    c->workspaces.push_back(w);
  }
  return RDKV_OK;
}

rdkv_status rdkv_cache_reserve_tail(rdkv_cache* c, int32_t max_new_tokens, void* stream) {
  if (!c) return fail(RDKV_ERR_INVALID_ARG, "cache is null");
  if (max_new_tokens <= 0) return fail(RDKV_ERR_INVALID_ARG, "max_new_tokens = %d must be positive", max_new_tokens);
  if (c->tail_cap != 0) return fail(RDKV_ERR_INVALID_ARG, "the tail of this cache is already reserved (%d tokens)", c->tail_cap);
  if (c->n_items == 0) { c->tail_cap = max_new_tokens; return RDKV_OK; }
  hipStream_t st = static_cast<hipStream_t>(stream);
  rdkv_status s = refuse_capture(st);
  if (s != RDKV_OK) return s;
  Allocator al{c->alloc, c->free_, c->alloc_user};
  const int64_t tail_tiles = (max_new_tokens + kTile64 - 1) / kTile64, tile_bytes = kTile64 * kHeadDim * 2;
  const int64_t side = c->n_items * tail_tiles * tile_bytes;     // K tiles of all items, then V tiles
  uint8_t* d_tail = static_cast<uint8_t*>(al.get(2 * side));
  if (!d_tail) return fail(RDKV_ERR_ALLOC, "device allocation failed");
  c->d_tail = d_tail;
  c->tail_cap = max_new_tokens;
  c->tail_len = 0;
  s = rebuild_schedule(c, d_tail, 2 * side, st);     // rows not yet appended must read as zeros
  if (s != RDKV_OK) {
    c->d_tail = nullptr;
    c->tail_cap = 0;
    al.put(d_tail);
  }
  return s;
}

rdkv_status rdkv_cache_append(rdkv_cache* c, const void* k_new, const void* v_new, void* stream) {
  if (!c || !k_new || !v_new) return fail(RDKV_ERR_INVALID_ARG, "cache, k_new and v_new must not be null");
  if (c->tail_cap == 0) return fail(RDKV_ERR_INVALID_ARG, "call rdkv_cache_reserve_tail before the first append");
  if (c->tail_len >= c->tail_cap)
    return fail(RDKV_ERR_INVALID_ARG, "the tail is full (%d tokens reserved)", c->tail_cap);
  if (c->n_items == 0) { c->tail_len += 1; return RDKV_OK; }
  RDKV_HIP(launch_append_rows(static_cast<const uint16_t*>(k_new), static_cast<const uint16_t*>(v_new), c->d_tail,
                              c->n_items, (c->tail_cap + kTile64 - 1) / kTile64, c->tail_cap, c->d_tail_len,
                              static_cast<hipStream_t>(stream)));
  c->tail_len += 1;
  return RDKV_OK;
}

int32_t rdkv_cache_tail_len(const rdkv_cache* c) { return c ? c->tail_len : 0; }

rdkv_status rdkv_cache_tail_len_sync(rdkv_cache* c, void* stream, int32_t* out) {
  if (!c) return fail(RDKV_ERR_INVALID_ARG, "cache is null");
  if (c->n_items > 0 && c->d_tail_len) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    const rdkv_status s = refuse_capture(st);
    if (s != RDKV_OK) return s;
    StageRegion r;
    int dev = 0;
    RDKV_HIP(stage_acquire(sizeof(int32_t), true, st, &r, &dev));
    CopyArgs a{};
    a.add(c->d_tail_len, r.data, sizeof(int32_t), kDstHost);
    RDKV_HIP(stage_round_trip(a, dev, r, st, [&] { std::memcpy(&c->tail_len, r.data, sizeof(int32_t)); }));
  }
  if (out) *out = c->tail_len;
  return RDKV_OK;
}

rdkv_status rdkv_cache_rebudget_tail(rdkv_cache* c, const rdkv_config* cfg, const void* Q_obs, void* stream) {
  if (!c || !cfg || !Q_obs) return fail(RDKV_ERR_INVALID_ARG, "cache, cfg and Q_obs must not be null");
  if (cfg->k_mode != c->k_mode || (c->k_mode == RDKV_K_CHANNELWISE && (cfg->k_scale_per_channel != 0) != (c->k_per_unit != 0)) ||
      cfg->group_size != c->group_size)
    return fail(RDKV_ERR_INVALID_ARG, "cfg must name the cache's own format (k_mode %d, k_scale_per_channel %d, group_size %d)",
                c->k_mode, c->k_per_unit, c->group_size);
  {   // appends replayed from a captured graph advance only the device's count: take that one
    const rdkv_status s0 = rdkv_cache_tail_len_sync(c, stream, nullptr);
    if (s0 != RDKV_OK) return s0;
  }
  if (c->tail_len <= 0) return fail(RDKV_ERR_INVALID_ARG, "no appended tokens to compress");
  if (cfg->batch != c->batch || cfg->hq != c->hq || cfg->hkv != c->hkv || cfg->head_dim != c->d)
    return fail(RDKV_ERR_SHAPE, "cfg (batch %d, hq %d, hkv %d, d %d) does not match the cache (%d, %d, %d, %d)",
                cfg->batch, cfg->hq, cfg->hkv, cfg->head_dim, c->batch, c->hq, c->hkv, c->d);
  if (!cfg->seq_lens) return fail(RDKV_ERR_INVALID_ARG, "seq_lens is null");
  for (int s = 0; s < cfg->batch; ++s)
    if (cfg->seq_lens[s] != c->tail_len)
      return fail(RDKV_ERR_SHAPE, "seq_lens[%d] = %d: every sequence has %d appended tokens", s, cfg->seq_lens[s], c->tail_len);
  {   // every host-side check of the pass comes before the first launch
    const rdkv_status s0 = check_config(cfg, true, true);
    if (s0 != RDKV_OK) return s0;
  }
  hipStream_t st = static_cast<hipStream_t>(stream);
  Allocator al{cfg->alloc, cfg->free_, cfg->alloc_user};
  Temp tmp(al, st);
  const int32_t n_tail = c->tail_len;
  const size_t elems = static_cast<size_t>(c->n_items) * n_tail * kHeadDim;
  tmp.reserve({elems * sizeof(uint16_t), elems * sizeof(uint16_t)});
  uint16_t* k_rows = tmp.get<uint16_t>(elems);
  uint16_t* v_rows = tmp.get<uint16_t>(elems);
  if (!k_rows || !v_rows) return fail(RDKV_ERR_ALLOC, "device allocation failed");
  RDKV_HIP(launch_gather_tail_rows(c->d_tail, c->n_items, (c->tail_cap + kTile64 - 1) / kTile64, n_tail, k_rows, v_rows, st));
  rdkv_cache* child = nullptr;
  rdkv_status s = rdkv_compress(cfg, k_rows, v_rows, Q_obs, stream, &child);   // synchronises the stream
  if (s != RDKV_OK) return s;
  // The tail's tiles keep the rows just compressed: rows at or past tail_len are masked out of the softmax (their
  // values are finite, so a zero probability times a stale V row adds nothing), and later appends overwrite them.
  c->absorbed.push_back(child);
  s = rebuild_schedule(c, c->d_tail_len, c->n_items * sizeof(int32_t), st);     // no token appended since
  if (s != RDKV_OK) {
    c->absorbed.pop_back();
    rdkv_cache_free(child);
    return s;
  }
  c->tail_len = 0;
  return RDKV_OK;
}

int32_t rdkv_cache_generations(const rdkv_cache* c) { return c ? static_cast<int32_t>(c->absorbed.size()) : 0; }

const rdkv_cache* rdkv_cache_generation(const rdkv_cache* c, int32_t index) {
  if (!c || index < 0 || index >= static_cast<int32_t>(c->absorbed.size())) return nullptr;
  return c->absorbed[index];
}

size_t rdkv_decode_bf16_workspace_bytes(const int32_t* seq_lens, int32_t batch, int32_t hq, int32_t hkv,
                                        int32_t head_dim) {
  if (check_shape(batch, hq, hkv, head_dim, seq_lens) != RDKV_OK || batch == 0) return 0;
  int chunk_rows, max_splits;
  dense_plan(seq_lens, batch, hkv, hq / hkv, &chunk_rows, &max_splits);
  const int64_t slots = static_cast<int64_t>(std::min(batch, kDenseMaxSeqs)) * hkv * max_splits;
  return static_cast<size_t>(slots) * (hq / hkv) * (kHeadDim + 2) * sizeof(float);
}

rdkv_status rdkv_decode_attn_bf16(const void* K, const void* V, const int32_t* seq_lens, int32_t batch, int32_t hq,
                                  int32_t hkv, int32_t head_dim, const void* q, float* out, float* lse,
                                  void* workspace, size_t workspace_bytes, void* stream) {
  rdkv_status s = check_shape(batch, hq, hkv, head_dim, seq_lens);
  if (s != RDKV_OK) return s;
  if (batch == 0) return RDKV_OK;
  if (!K || !V || !q || !out || !workspace) return fail(RDKV_ERR_INVALID_ARG, "K, V, q, out, workspace must not be null");
  const size_t need = rdkv_decode_bf16_workspace_bytes(seq_lens, batch, hq, hkv, head_dim);
  if (workspace_bytes < need)
    return fail(RDKV_ERR_INVALID_ARG, "workspace of %zu bytes is smaller than the %zu required", workspace_bytes, need);
  const int g = hq / hkv;
  int chunk_rows, max_splits;
  dense_plan(seq_lens, batch, hkv, hq / hkv, &chunk_rows, &max_splits);
  const int64_t slots = static_cast<int64_t>(std::min(batch, kDenseMaxSeqs)) * hkv * max_splits;
  const size_t heads = static_cast<size_t>(batch) * hq;
  size_t rows = 0;
  for (int i = 0; i < batch; ++i) rows += static_cast<size_t>(seq_lens[i]) * hkv;
  const size_t row = kHeadDim * sizeof(uint16_t);
  const bool apart = dense_outputs_apart({K, rows * row}, {V, rows * row}, {q, heads * row}, {out, heads * kHeadDim * sizeof(float)},
                                         {lse, lse ? heads * sizeof(float) : 0});
  const bool together = apart && dense_together(seq_lens, batch, hkv, g, max_splits);
  int64_t row_off = 0;
  for (int s0 = 0; s0 < batch; s0 += kDenseMaxSeqs) {
    const int ns = std::min(kDenseMaxSeqs, batch - s0);
    DenseArgs a;
    a.K = static_cast<const uint16_t*>(K);
    a.V = static_cast<const uint16_t*>(V);
    a.q = static_cast<const uint16_t*>(q);
    a.part_acc = static_cast<float*>(workspace);
    a.part_ml = a.part_acc + slots * g * kHeadDim;
    a.out = out;
    a.lse = lse;
    a.hq = hq; a.hkv = hkv; a.batch = batch; a.chunk_rows = chunk_rows; a.max_splits = max_splits; a.seq_base = s0;
    a.tag[0] = a.tag[1] = 0;
    if (together) next_tag(a.tag);
    for (int i = 0; i < ns; ++i) {
      a.T[i] = seq_lens[s0 + i];
      a.row_off[i] = row_off;
      row_off += static_cast<int64_t>(seq_lens[s0 + i]) * hkv;
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    {
      TimedScope ts(RDKV_TIME_DECODE_BF16, st);
      RDKV_HIP(launch_decode_dense_split(a, g, ns, st));
    }
    if (!together) RDKV_HIP(launch_decode_dense_merge(a, g, ns, st));
  }
  return RDKV_OK;
}

}  // extern "C"

// ---- the bf16 decode step for callers that cannot allocate ---------------------------------------------------------
// Its split partials live in a file-scope device array instead of a caller workspace.  In host code the array's name
// is only a stand-in for the symbol: the device address is looked up once per device and used from then on.
constexpr size_t kStaticScratchBytes = static_cast<size_t>(8) << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device (looked up on the first call on that device).
rdkv_status static_scratch(void** out) {
  int dev = -1;
  RDKV_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return fail(RDKV_ERR_UNSUPPORTED, "device index %d out of range", dev);
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    RDKV_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return fail(RDKV_ERR_HIP, "hipGetSymbolAddress returned a null address");
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return RDKV_OK;
}
}  // namespace

extern "C" {

size_t rdkv_decode_bf16_noalloc_max_bytes(void) { return kStaticScratchBytes; }

rdkv_status rdkv_decode_attn_bf16_noalloc(const void* K, const void* V, const int32_t* seq_lens, int32_t batch,
                                          int32_t hq, int32_t hkv, int32_t head_dim, const void* q, float* out,
                                          float* lse, void* stream) {
  rdkv_status s = check_shape(batch, hq, hkv, head_dim, seq_lens);
  if (s != RDKV_OK) return s;
  if (batch == 0) return RDKV_OK;
  const size_t need = rdkv_decode_bf16_workspace_bytes(seq_lens, batch, hq, hkv, head_dim);
  if (need > kStaticScratchBytes)
    return fail(RDKV_ERR_UNSUPPORTED,
                "this batch needs %zu bytes of split partials, more than the %zu bytes of the built-in scratch area; "
                "use rdkv_decode_attn_bf16 with a workspace",
                need, kStaticScratchBytes);
  void* ws = nullptr;
  s = static_scratch(&ws);
  if (s != RDKV_OK) return s;
  // every partial slot the merge reads is written by the split kernel of the same call: nothing to clear
  return rdkv_decode_attn_bf16(K, V, seq_lens, batch, hq, hkv, head_dim, q, out, lse, ws, kStaticScratchBytes, stream);
}

rdkv_status rdkv_cache_stats(const rdkv_cache* c, rdkv_stats* out) {
  if (!c || !out) return fail(RDKV_ERR_INVALID_ARG, "cache and out must not be null");
  std::memset(out, 0, sizeof(*out));
  out->n_items = c->n_items;
  int64_t kept = 0;
  for (int64_t i = 0; i < c->n_items; ++i)
    for (int ti = 0; ti < 4; ++ti) {
      const int bits = pack_tier_bits(ti);
      const int64_t cnt = c->counts[i * 4 + ti];
      out->rows[ti] += cnt;
      kept += cnt;
      (void)bits;
    }
  out->stored_bytes = c->stored_bytes;
  out->evicted = c->total_tokens - kept;
  out->arena_bytes = c->arena_bytes;
  out->index_bytes = c->index_bytes;
  out->n_chunks = static_cast<int64_t>(c->chunks.size()) - c->n_cont;   // launched work items (not their continuations)
  out->dense_bytes = c->total_tokens * kHeadDim * 2 * 2;
  out->lambda_min = out->lambda_max = std::nan("");
  if (c->d_lambda && c->d_iters && c->n_items > 0) {   // the token map's searches (Alg. 2); synchronous copies
    std::vector<double> lam(c->n_items);
    std::vector<int32_t> iters(c->n_items);
    RDKV_HIP(hipMemcpy(lam.data(), c->d_lambda, lam.size() * sizeof(double), hipMemcpyDeviceToHost));
    RDKV_HIP(hipMemcpy(iters.data(), c->d_iters, iters.size() * sizeof(int32_t), hipMemcpyDeviceToHost));
    out->alloc_info = 1;
    for (int64_t i = 0; i < c->n_items; ++i) {
      out->iterations_max = std::max<int64_t>(out->iterations_max, iters[i]);
      if (std::isnan(lam[i])) continue;
      out->lambda_min = std::isnan(out->lambda_min) ? lam[i] : std::min(out->lambda_min, lam[i]);
      out->lambda_max = std::isnan(out->lambda_max) ? lam[i] : std::max(out->lambda_max, lam[i]);
    }
  }
  for (const rdkv_cache* child : c->absorbed) {   // appended tokens compressed later count like the prompt's
    rdkv_stats cs;
    rdkv_cache_stats(child, &cs);
    for (int ti = 0; ti < 4; ++ti) out->rows[ti] += cs.rows[ti];
    out->evicted += cs.evicted;
    out->stored_bytes += cs.stored_bytes;
    out->arena_bytes += cs.arena_bytes;
    out->index_bytes += cs.index_bytes;
    out->n_chunks += cs.n_chunks;
    out->dense_bytes += cs.dense_bytes;
  }
  return RDKV_OK;
}

int32_t rdkv_k_row_words(const uint8_t* bits_ch) {
  if (!bits_ch || !valid_map(bits_ch)) return -1;
  int32_t held[4];
  return make_item_k(bits_ch, held).n_words_padded;
}

int32_t rdkv_k_row_words_max(void) { return kMaxKRowWords; }

// Not part of the interface: how often the merging workgroups of this cache's decode launches look before they leave their
// blocks to the chunks.  A test's way to have them give up at once.
void rdkv_cache_set_looks(rdkv_cache* c, int32_t looks) { c->looks = looks; }

size_t rdkv_cache_export_bytes(const rdkv_cache* c, int what) {
  if (!c) return 0;
  switch (what) {
    case RDKV_EXPORT_COUNTS: return c->counts.size() * sizeof(int32_t);
    case RDKV_EXPORT_TIER_IDX: return static_cast<size_t>(c->kept_total) * sizeof(int32_t);
    case RDKV_EXPORT_SEG_OFF: return c->seg_off.size() * sizeof(int64_t);
    case RDKV_EXPORT_ARENA: return static_cast<size_t>(c->arena_bytes);
    case RDKV_EXPORT_BITS_TOK: return static_cast<size_t>(c->total_tokens);
    case RDKV_EXPORT_BITS_CH: return c->d_bits_ch ? static_cast<size_t>(c->n_items) * kHeadDim : 0;
    case RDKV_EXPORT_LAMBDA:
      return c->d_lambda ? static_cast<size_t>(c->n_items) * (c->k_mode == RDKV_K_CHANNELWISE ? 2 : 1) * sizeof(double) : 0;
    case RDKV_EXPORT_ITERATIONS:
      return c->d_iters ? static_cast<size_t>(c->n_items) * (c->k_mode == RDKV_K_CHANNELWISE ? 2 : 1) * sizeof(int32_t) : 0;
    default: return 0;
  }
}

rdkv_status rdkv_cache_export(const rdkv_cache* c, int what, void* dst, size_t bytes) {
  if (!c || (!dst && bytes > 0)) return fail(RDKV_ERR_INVALID_ARG, "cache and dst must not be null");
  const size_t need = rdkv_cache_export_bytes(c, what);
  if (what < RDKV_EXPORT_COUNTS || what > RDKV_EXPORT_ITERATIONS) return fail(RDKV_ERR_INVALID_ARG, "unknown export %d", what);
  if (bytes < need) return fail(RDKV_ERR_INVALID_ARG, "destination of %zu bytes is smaller than the %zu required", bytes, need);
  if (need == 0) return RDKV_OK;
  switch (what) {
    case RDKV_EXPORT_COUNTS: std::memcpy(dst, c->counts.data(), need); break;
    case RDKV_EXPORT_SEG_OFF: std::memcpy(dst, c->seg_off.data(), need); break;
    case RDKV_EXPORT_TIER_IDX: RDKV_HIP(hipMemcpy(dst, c->d_tier_idx, need, hipMemcpyDeviceToHost)); break;
    case RDKV_EXPORT_ARENA: RDKV_HIP(hipMemcpy(dst, c->d_arena, need, hipMemcpyDeviceToHost)); break;
    case RDKV_EXPORT_BITS_TOK: RDKV_HIP(hipMemcpy(dst, c->d_bits_tok, need, hipMemcpyDeviceToHost)); break;
    case RDKV_EXPORT_BITS_CH: RDKV_HIP(hipMemcpy(dst, c->d_bits_ch, need, hipMemcpyDeviceToHost)); break;
    case RDKV_EXPORT_LAMBDA: RDKV_HIP(hipMemcpy(dst, c->d_lambda, need, hipMemcpyDeviceToHost)); break;
    case RDKV_EXPORT_ITERATIONS: RDKV_HIP(hipMemcpy(dst, c->d_iters, need, hipMemcpyDeviceToHost)); break;
  }
  return RDKV_OK;
}

void rdkv_cache_free(rdkv_cache* c) {
  if (!c) return;
  free_cache_buffers(c);
  if (!c->alloc)
    if (ScratchPool* pool = scratch_pool()) pool->give_back();
  delete c;
}

}  // extern "C"
