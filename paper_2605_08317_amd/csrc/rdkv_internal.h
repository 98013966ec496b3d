// Internal declarations shared by the host side of librdkv and its kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <mutex>
#include <string>
#include <vector>

#include "rdkv.h"

namespace rdkv {

constexpr int kHeadDim = 128;
constexpr int kGroup = 32;             // quantization group (channels)
constexpr int kGroupsPerRow = kHeadDim / kGroup;
constexpr int kMostChunkRows = 1 << 21;   // of a chunk of the decode schedule: a side of it is smaller than 2^30 bytes
constexpr int kTile64 = 64;            // tier segments are padded to whole 64-row tiles
constexpr int kKTokenGroup = 32;       // mixed mode: a K channel's group = 32 consecutive retained tokens of a segment
constexpr int kPartBlock = 1024;       // tokens per block of the tier counts
constexpr int kKeyTile = 64;           // keys per tile of the weights kernels
constexpr int kSegAlign = 256;         // byte alignment of arena segments
constexpr int kNumPackTiers = 4;       // stored tiers, order 16, 8, 4, 2
constexpr int kDenseMaxSeqs = 64;      // sequences per dense-decode launch (kernel-argument table)

__host__ __device__ inline int pack_tier_bits(int ti) { return 16 >> ti; }          // 0..3 -> 16,8,4,2
__host__ __device__ inline int tier_row_bytes(int bits) { return kHeadDim * bits / 8; }
__host__ __device__ inline int tier_meta_bytes(int bits) { return bits == 16 ? 0 : kGroupsPerRow * 4; }

// One unit of decode work: a run of rows of one tier of one item.
struct Chunk {
  int64_t k_data, k_meta, v_data, v_meta;   // byte offsets into the arena
  int32_t rows;                             // valid rows in this chunk
  int32_t tier;                             // 16, 8, 4, 2, kTierTail, kTierMerge
  int32_t item;                             // sequence * hkv + kv head
  int32_t slot;                             // partial-result slot
  int16_t k_word_end[4];                    // mixed mode: ItemK::word_end of the item (the shape of its K rows)
  int32_t row0;                             // appended-token zone: first row of the chunk inside the item's tail;
                                            // kTierMerge: which of the item's merging workgroups
  int32_t reserved;                         // mixed mode: index of the chunk's ItemK in the schedule's table
                                            // (generation * items + item)
  int32_t slot0, nslots;                    // the item's first partial slot and its number of slots (= chunks)
  int32_t next;                             // token-wise quantized tiers: index in the chunk table of the piece the same
                                            // workgroup goes on with (another tier of the same item), -1: none
  int32_t pad_;
};
constexpr int kTailChunkRows = 256;         // appended tokens per decode work item
constexpr int kTierTail = 17;               // Chunk::tier of a chunk of appended tokens (64-token tiles of bf16 rows)
constexpr int kTierMerge = 18;              // Chunk::tier of a workgroup that merges an item's partials (decode_merge.h)

// Channel-wise K (mixed mode): how one item's K tiles are laid out.  Channels are sorted by bit-width into
// slots: tiers 16, 8, 4, 2 in this order.  A retained token's K row is a run of 32-bit words (a 16-bit word holds
// 2 slots, an 8-bit word 4, a 4-bit word 8, a 2-bit word 16); every tier is padded to whole words, the 16-bit tier
// to whole word pairs, the row to an even number of words.  A step is 4 consecutive slots.
constexpr int kMaxSlots = 160;   // 128 channels + up to 3 + 3 + 7 + 15 padding slots
constexpr int kMaxKRowWords = 68;  // longest row: 125 channels at 16 bits, one each at 8, 4, 2 -> 64 + 1 + 1 + 1, evened
struct ItemK {
  int32_t kt_bytes;              // K tile (64 tokens) data bytes = 256 * n_words_padded
  int32_t km_bytes;              // K tile metadata bytes = 32 * n_qsteps (2 token groups x 16 bytes per quantized step)
  int16_t word_end[4];           // words per token up to and including tier 16, 8, 4, 2
  int16_t slot_base[4];          // first slot of each tier
  int16_t n_slots, n_words, n_words_padded;
  int16_t n_steps16, n_qsteps;   // steps of the 16-bit tier; steps of the quantized tiers
  int16_t slot_ch[kMaxSlots];    // channel held by a slot, -1 for padding
};

// What the kernels of a compression pass need to know about a batch, an entry per sequence.  Up to kSeqsAlong of them come
// with every launch, in its arguments: no launch has to bring a table to the device first, and a kernel's first loads wait for
// the entries alone.  More of them are a table in device memory.  (1 KB of arguments costs the host 0.1 us a launch, a launch that
// copies a table 2.4 and the device 3.3: staged calls on 50K keys 196.5 -> 189.5 us, compressing 4K keys 54.4 -> 52.6.)
struct SeqEntry {
  int64_t row0;                  // first token of the sequence in ragged [hkv][T] arrays
  int32_t T, tile0, blk0;        // tokens; first key tile and first block of the bit map of the sequence's items
  float avg, budget;             // average bits per cache element, and of the token map (channel-wise mode: the V share)
  int32_t pad_;
};
constexpr int kSeqsAlong = 32;
struct Batch {
  const SeqEntry* table;         // device memory, or null: own
  int32_t n_seqs, hkv;
  uint32_t inv_hkv;              // 2^32 / hkv, rounded up (2^32 - 1 for one head)
  SeqEntry own[kSeqsAlong];
  // (constant address space, as the arguments' is: one scalar load whichever of the two it comes from)
  typedef const __attribute__((address_space(4))) SeqEntry* ConstEntries;
  __device__ __forceinline__ SeqEntry seq(int s) const {
    if (!table) return own[s];
    const ConstEntries t = (ConstEntries)(table) + s;
    return SeqEntry{t->row0, t->T, t->tile0, t->blk0, t->avg, t->budget, 0};
  }
  __device__ __forceinline__ int tile0(int s) const { return table ? table[s].tile0 : own[s].tile0; }
};
// one item = (sequence, KV head)
struct ItemOf {
  int seq, head, T, tile0, blk0;
  int64_t off;                   // first token
  double avg, budget;
  __device__ __forceinline__ ItemOf(const Batch& b, int item) {
    seq = static_cast<int>(__umulhi(static_cast<uint32_t>(item), b.inv_hkv));      // off by one at most
    head = item - seq * b.hkv;
    if (head < 0) {
      --seq;
      head += b.hkv;
    } else if (head >= b.hkv) {
      ++seq;
      head -= b.hkv;
    }
    const SeqEntry e = b.seq(seq);
    T = e.T;
    off = e.row0 + static_cast<int64_t>(head) * e.T;
    tile0 = e.tile0 + head * tiles();
    blk0 = e.blk0 + head * ((e.T + kPartBlock - 1) / kPartBlock);
    avg = static_cast<double>(e.avg);
    budget = static_cast<double>(e.budget);
  }
  __device__ __forceinline__ int tiles() const { return (T + kKeyTile - 1) / kKeyTile; }
};

// Slots of a tier of a K row with n channels (ItemK): whole word pairs of 16-bit slots, whole words of the others.
__host__ __device__ inline uint32_t k_tier_slots(int ti, uint32_t n) {
  const uint32_t pad = ti == 0 ? 4u : 2u << ti;
  return (n + pad - 1u) & ~(pad - 1u);
}
// Bytes of a 64-row tile of channel-wise K: its codes (words: of a row, padded to an even number), its scales and offsets (steps:
// quantized steps of four slots; a record per group of kKTokenGroup rows).
__host__ __device__ inline int32_t k_tile_bytes(int words) { return 4 * kTile64 * words; }
__host__ __device__ inline int32_t k_meta_bytes(int steps) { return kTile64 / kKTokenGroup * 16 * steps; }
// Sizes of the four segments of a tier of an item -- K codes, K scales and offsets, V codes, V scales and offsets, one behind the
// other in the arena -- in units of kSegAlign bytes.  The host's plan (the chunk table, the arena's size) and the device's (where the
// packing kernels write) both come from here.  words, steps: of a channel-wise K row; token-wise K: words 0.
struct SegmentUnits { uint64_t k_data, k_meta, v_data, v_meta; };
__host__ __device__ inline SegmentUnits segment_units(int ti, uint64_t rows, bool channelwise, int words, int steps, bool per_unit) {
  const int bits = 16 >> ti;
  const uint64_t tiles = (rows + kTile64 - 1) / kTile64;
  static_assert(kTile64 * kHeadDim / 8 % kSegAlign == 0 && kTile64 * kGroupsPerRow * 4 % kSegAlign == 0 && 4 * kTile64 % kSegAlign == 0,
                "whole units a tile");
  SegmentUnits u;
  u.v_data = tiles * static_cast<uint32_t>(kTile64 * tier_row_bytes(bits) / kSegAlign);
  u.v_meta = tiles * static_cast<uint32_t>(kTile64 * tier_meta_bytes(bits) / kSegAlign);
  if (!channelwise) {
    u.k_data = u.v_data;
    u.k_meta = u.v_meta;
    return u;
  }
  u.k_data = tiles * static_cast<uint32_t>(k_tile_bytes(words) / kSegAlign);
  const uint64_t meta = per_unit ? (rows > 0 ? static_cast<uint32_t>(k_meta_bytes(steps) / (kTile64 / kKTokenGroup)) : 0u)      // one record
                                 : tiles * static_cast<uint32_t>(k_meta_bytes(steps));
  u.k_meta = (meta + kSegAlign - 1) / kSegAlign;
  return u;
}
// Device tables that one workgroup of the launch with the position lists makes for the packing kernels, so that these wait for
// nothing that the host makes.
struct PlanArgs {
  int64_t* idx_base;             // [items][4]: first of a tier's kept positions
  int64_t* seg_off;              // [items][4][4]: arena offsets
  int32_t* counts;               // [items][4]: rows per tier
  const uint8_t* bits_ch;        // [items][128] channel-wise K, or null
  ItemK* items_k;                // [items] channel-wise K, or null
  int32_t n_items, per_unit;     // per_unit: one K scale per channel
};

// Lets a kernel use more dynamic LDS than the runtime grants by default; asked once per kernel and device (a call costs
// 0.5 us).
template <class K>
inline hipError_t allow_lds(K kernel, size_t lds, std::atomic<uint64_t>* asked) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = 1ull << (dev & 63);
  if (asked->load(std::memory_order_relaxed) & bit) return hipSuccess;
  e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
  if (e == hipSuccess) asked->fetch_or(bit, std::memory_order_relaxed);
  return e;
}
// `most`: the most the kernel is ever launched with
#define RDKV_ALLOW_LDS(kernel, most)                        \
  [&]() -> hipError_t {                                     \
    static std::atomic<uint64_t> asked{0};                  \
    return rdkv::allow_lds(kernel, most, &asked);           \
  }()

// One launch of small copies (copy_kernels.hip).  Segments with a side in staging memory are added first.
constexpr int kCopySegs = 9;
constexpr int kStageWords = 16;        // completion words at the head of a staging region
enum : int32_t { kSrcHost = 1, kDstHost = 2 };
struct CopySeg {
  const void* src;                     // null: fill with the two words of `fill`
  void* dst;
  int64_t bytes;
  uint32_t fill[2];
  int32_t side;                        // kSrcHost or kDstHost: that side is staging memory; 0: both are device memory
};
struct CopyArgs {
  int32_t n;
  int32_t first[kCopySegs + 1];        // first workgroup of a segment (plan_copy)
  uint32_t* words;                     // completion words of the staging region, or null
  uint32_t seq;
  int32_t host_blocks;                 // workgroups that set a word (plan_copy)
  CopySeg seg[kCopySegs];
  void add(const void* src, void* dst, int64_t bytes, int32_t side = 0) {
    if (bytes > 0) seg[n++] = CopySeg{src, dst, bytes, {0u, 0u}, side};
  }
  void fill(void* dst, int64_t bytes, uint32_t w0, uint32_t w1) {
    if (bytes > 0) seg[n++] = CopySeg{nullptr, dst, bytes, {w0, w1}, 0};
  }
};
void plan_copy(CopyArgs& a);           // after the last segment, before launch_copy
hipError_t launch_copy(const CopyArgs& a, hipStream_t st);
// The same for a stream under capture: segments out of host memory only, whose bytes the recorded launches carry themselves.
hipError_t launch_copy_by_value(const CopyArgs& a, hipStream_t st);

// What the search's kernels leave for the host in staging memory by themselves: words of (tag, value), and the host watches
// each.  Null: nobody waits.
struct CountPost {
  uint64_t* counts;                    // [items][4]: units in tiers 16, 8, 4, 2
  uint64_t* channels;                  // [items][4 tiers][4]: which of 32 channels each have the tier's width
  uint32_t tag;
};

struct DenseArgs {
  const uint16_t* K;
  const uint16_t* V;
  const uint16_t* q;
  float* part_acc;     // [slots][g][128]
  float* part_ml;      // [slots][g][2]
  float* out;
  float* lse;
  int32_t hq, hkv, batch, chunk_rows, max_splits, seq_base;
  uint32_t tag[2];     // of this launch, which merges its own partials; or zeros: a merge launch follows
  int32_t T[kDenseMaxSeqs];
  int64_t row_off[kDenseMaxSeqs];           // first row of the sequence block in K / V
};

// ---- launchers implemented in the .hip files ------------------------------
hipError_t launch_decode_dense_split(const DenseArgs& a, int g, int n_seqs, hipStream_t st);
hipError_t launch_decode_dense_merge(const DenseArgs& a, int g, int n_seqs, hipStream_t st);
struct MergeArgs;   // decode_merge.h
// 16-bit tier of a token-wise cache (row-major bf16 rows)
hipError_t launch_decode_tiered_split(const Chunk* chunks, int n_chunks, const uint8_t* arena, const uint16_t* q,
                                      const MergeArgs& ma, hipStream_t st);
// tail_len: the cache's device words, appended tokens so far of every item (equal for all)
hipError_t launch_append_rows(const uint16_t* k_new, const uint16_t* v_new, uint8_t* tail, int64_t n_items,
                              int32_t tail_tiles, int32_t tail_cap, int32_t* tail_len, hipStream_t st);
hipError_t launch_gather_tail_rows(const uint8_t* tail, int64_t n_items, int32_t tail_tiles, int32_t n,
                                   uint16_t* k_rows, uint16_t* v_rows, hipStream_t st);

// chunks: the whole chunk table; workgroup b starts with chunks[first + b] and, if `multi`, follows Chunk::next.
// ma.parts > 0: the partials are looked for, by the n_merge entries of tier kTierMerge behind the n_chunks; otherwise arrivals
// are counted.  The former, and a range that starts with chunks of the 16-bit tier (rows16), only where decode_tiles_take_rows
// says so.
// tail_len: device word holding the appended tokens that exist so far (chunks of tier kTierTail end there)
bool decode_tiles_take_rows(int n_chunks, bool multi);
hipError_t launch_decode_tiles(const Chunk* chunks, int first, int n_chunks, int n_merge, bool rows16, bool multi,
                               const uint8_t* arena, const uint16_t* q, const MergeArgs& ma, const int32_t* tail_len, hipStream_t st);
// one object per head-set count (hs1: up to 4 query heads per KV head, hs2: 8)
// One object per head-set count (hs1: up to 4 query heads per KV head, hs2: 8) and row length class (long0: K rows
// of up to 32 words, long1: up to 68).  waves: wavefronts per workgroup, 4 or 8 (8 only in hs1 / long0).
#define RDKV_DECLARE_MIXED(NAME_)                                                                                \
  hipError_t NAME_(const Chunk* chunks, int n_chunks, const uint8_t* arena, const ItemK* items_k, int max_words, \
                   int max_steps, int max_qsteps, const uint16_t* q, const MergeArgs& ma, const int32_t* tail_len, \
                   int per_unit, int waves, hipStream_t st);
RDKV_DECLARE_MIXED(launch_decode_mixed_hs1_long0)
RDKV_DECLARE_MIXED(launch_decode_mixed_hs1_long1)
RDKV_DECLARE_MIXED(launch_decode_mixed_hs2_long0)
RDKV_DECLARE_MIXED(launch_decode_mixed_hs2_long1)
#undef RDKV_DECLARE_MIXED
inline hipError_t launch_decode_mixed(const Chunk* chunks, int n_chunks, const uint8_t* arena, const ItemK* items_k,
                                      int max_words, int max_steps, int max_qsteps, const uint16_t* q,
                                      const MergeArgs& ma, const int32_t* tail_len, int per_unit, int waves,
                                      hipStream_t st);

// Optional event bracketing of the main kernels (rdkv_kernel_timing_*).
void timing_begin(int kind, hipStream_t st);
void timing_end(int kind, hipStream_t st);
struct TimedScope {
  int kind;
  hipStream_t st;
  TimedScope(int k, hipStream_t s) : kind(k), st(s) { timing_begin(kind, st); }
  ~TimedScope() { timing_end(kind, st); }
};

}  // namespace rdkv

// The opaque handle of the C ABI.
struct rdkv_cache {
  int32_t batch = 0, hq = 0, hkv = 0, d = 0, k_mode = 0;
  int32_t k_per_unit = 0;               // mixed mode: one K scale per channel over all retained tokens (App. B)
  int32_t group_size = 32;              // channels per scale of a token row: 32, or 128 = one scale per row (App. B)
  std::vector<int32_t> seq_lens;
  int64_t n_items = 0;
  int64_t total_tokens = 0;             // sum_s hkv * T_s
  // host copies
  std::vector<int32_t> counts;          // [items][4]
  std::vector<int64_t> seg_off;         // [items][4][4]
  std::vector<rdkv::Chunk> chunks;
  int64_t arena_bytes = 0;
  int64_t kept_total = 0;
  int64_t n_chunks16 = 0;               // leading chunks of the 16-bit tier
  // device memory (owned): rdkv_pack takes one block for the arena and every table below; what later calls add or
  // replace (tail, rebuilt chunk tables, workspaces of other streams) are allocations of their own
  uint8_t* d_block = nullptr;
  int64_t block_bytes = 0;
  uint8_t* d_arena = nullptr;
  int32_t* d_tier_idx = nullptr;        // [kept_total]
  rdkv::Chunk* d_chunks = nullptr;
  // split workspaces, one per stream that has decoded from this cache: partial results (decode_merge.h) and the items' arrival counters (zero between steps)
  struct Workspace {
    hipStream_t stream;
    float* part_acc;
    float* part_ml;
    int32_t* arrive;
    void* block;                        // the one allocation behind the three
  };
  mutable std::vector<Workspace> workspaces;
  mutable std::mutex ws_mu;
  int64_t n_slots = 0;                  // partial slots of the whole schedule
  int32_t* d_tail_len = nullptr;        // [items]: appended tokens so far (equal for all)
  int32_t mixed_waves = 4;              // channel-wise mode: wavefronts per workgroup of the decode kernel (4 or 8)
  uint8_t* d_bits_tok = nullptr;        // copy of the token bit map
  uint8_t* d_bits_ch = nullptr;         // [items][128] K channel bit map (mixed mode)
  rdkv::ItemK* d_items_k = nullptr;     // [items] (mixed mode)
  std::vector<rdkv::ItemK> items_k;
  int32_t max_k_words = 0, max_k_steps = 0, max_k_qsteps = 0;   // largest K row shape over the items (mixed mode)
  // appended-token zone (Zone C): per item ceil(tail_cap / 64) tiles of 64 bf16 K rows (16 KiB each), then the same
  // for V, in one allocation (zero-filled: rows not yet appended read as zeros)
  std::vector<int32_t> slot_begin, slot_count;   // host copies of the partial-slot tables
  uint8_t* d_tail = nullptr;
  int64_t n_merge = 0;                  // merging workgroups of the schedule, behind the launched chunks in d_chunks
  int32_t merge_parts = 0;              // MergeArgs::parts
  int32_t looks = 256;                  // MergeArgs::looks: a look takes 1 us, a launch that looks at most 50
  int64_t n_tail_chunks = 0;            // chunks of the tail, appended to d_chunks in (chunk index, item) order:
                                        // the first ceil(tail_len / 256) * items of them are live
  int32_t tail_cap = 0, tail_len = 0;
  // streaming re-budgeting: appended tokens that were compressed later, one packed cache per call (owned); their
  // chunks are part of this cache's decode schedule (d_chunks), with offsets relative to d_arena
  std::vector<rdkv_cache*> absorbed;
  std::vector<int32_t> own_slot_count;  // [items]: partial slots of this cache's own chunks (no tail, no absorbed)
  int64_t sched16 = 0, schedq = 0;      // chunks of the schedule: 16-bit tier, then the quantized tiers (all generations)
  int64_t n_cont = 0;                   // continuation pieces of this cache's own chunks: the last n_cont entries of `chunks`
  rdkv::ItemK* d_items_sched = nullptr; // mixed mode with absorbed generations: [generations][items] K row layouts
  int32_t sched_k_words = 0, sched_k_steps = 0, sched_k_qsteps = 0;   // largest K row shape over all generations
  double* d_lambda = nullptr;           // [items] (token map), channel-wise mode: + [items] (channel map): the
  int32_t* d_iters = nullptr;           // multiplier and the step count of every search (rdkv_compress only)
  int64_t stored_bytes = 0;             // bytes a decode step must read (unpadded)
  int64_t index_bytes = 0;
  rdkv_alloc_fn alloc = nullptr;
  rdkv_free_fn free_ = nullptr;
  void* alloc_user = nullptr;
};
