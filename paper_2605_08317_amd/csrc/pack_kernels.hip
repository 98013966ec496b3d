// Stage 4 of Alg. 1 on the GPU: stable per-tier partition of the token bit map and
// group-wise quantize-and-pack into tier segments (16-bit rows row-major, quantized tiers in 64-row tiles in
// token-wise mode and 32-row tiles in mixed mode).
//
// The quantizer is fp32 in a fixed operation order (this file is compiled with
// floating-point contraction off) so that codes, scales and offsets are
// reproducible bit for bit:
//   mn = min x, mx = max x            over a group of 32 channels
//   s  = fp16_rn((mx - mn) / Q)        Q = 2^b - 1, IEEE divide
//   m  = fp16_rn(mn)
//   code = clamp(rint((x - m) / s), 0, Q), all zero when s == 0; the quotient is the correctly rounded one, from the
//          hardware reciprocal of s and one exact remainder (see Quant::code)
// Codes occupy b-bit fields of little-endian words (App. B: fields at bit offsets 0,2,4,6 / 0,4 of a byte).
#include <algorithm>
#include <type_traits>

#include "copy_device.h"
#include "wave_ops.h"

namespace rdkv {

namespace {

__device__ __forceinline__ int tier_slot(uint8_t b) {   // 16,8,4,2 -> 0..3 ; else -1
  return b == 16 ? 0 : b == 8 ? 1 : b == 4 ? 2 : b == 2 ? 3 : -1;
}

// four bytes of a bit map at any address
struct __attribute__((packed, aligned(1))) Bytes4 { uint32_t v; };

// Counts of each stored tier inside every block of 1024 tokens of every item; a first count of -1: the block holds a value
// that is no bit-width.
__global__ __launch_bounds__(256) void tier_count_kernel(const uint8_t* __restrict__ bits, int4* __restrict__ blk_counts,
                                                         Batch batch) {
  __shared__ int s_cnt[4][5];
  const ItemOf it(batch, blockIdx.y);
  const int T = it.T;
  const int t0 = blockIdx.x * kPartBlock;
  if (t0 >= T) return;
  const int tid = threadIdx.x, wave = tid >> 6;
  const uint8_t* b = bits + it.off + t0;
  const int n = min(kPartBlock, T - t0), u = 4 * tid;
  uint32_t four = 0;
  if (u + 3 < n) four = reinterpret_cast<const Bytes4*>(b + u)->v;
  else
    for (int e = 0; e < 4; ++e)
      if (u + e < n) four |= static_cast<uint32_t>(b[u + e]) << (8 * e);
  int c[5] = {0, 0, 0, 0, 0};            // the four tiers, and what is neither a tier nor 0 (evicted)
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const uint8_t v = static_cast<uint8_t>(four >> (8 * e));
    const int s = tier_slot(v);
#pragma unroll
    for (int k = 0; k < 4; ++k) c[k] += __popcll(__ballot(s == k));
    c[4] += __popcll(__ballot(s < 0 && v != 0));
  }
  if ((tid & 63) == 0)
#pragma unroll
    for (int k = 0; k < 5; ++k) s_cnt[wave][k] = c[k];
  __syncthreads();
  if (tid == 0) {
    int sum[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) sum[k] = s_cnt[0][k] + s_cnt[1][k] + s_cnt[2][k] + s_cnt[3][k];
    blk_counts[it.blk0 + blockIdx.x] = make_int4(sum[4] > 0 ? -1 : sum[0], sum[1], sum[2], sum[3]);
  }
}

// One launch between the bit map and the packing; nothing in it needs the host:
//   - the ascending position lists of every tier, item by item in scratch: item's first token + kept tokens of the higher
//     tiers + rank (one workgroup = one block of 1024 tokens, a thread = four consecutive ones; the ranks of all four tiers
//     come from one prefix sum over 16-bit fields)
//   - the counts' way to the host, who waits for them and so for this launch, unless the search has posted them (CountPost: compressing
//     items of up to 32K tokens), and what else is copied or filled then (copy_part)
//   - the arena's plan (plan_part), by one workgroup
//   - channel-wise K: the row layout of every item (layout_part), by the item's first workgroup
// What bounds it is latency: two round trips to memory and the launch (4.4 us for two items of 4K tokens, 9.3 for 128 of 20K).
// With the counts copied by a launch in front of the wait, and the tables and then the lists in two launches behind it,
// compressing two heads of 4K keys took 58.0 us, eight of 128K 242; now 53.2 and 234.
struct ScatterArgs {
  const uint8_t* bits;
  const int4* blk_counts;
  int32_t* tier_idx;
  int32_t extra;                 // leading workgroups of every grid row that do other things
  PlanArgs plan;
  CopyArgs copy;
  Batch batch;
};

// counts of a block; one that holds a value that is no bit-width (the host refuses the map) counts as empty there
__device__ __forceinline__ int4 block_counts(const int4* blk_counts, int b) {
  int4 c = blk_counts[b];
  c.x = max(c.x, 0);
  return c;
}

// Sum over groups of 2^k consecutive lanes, in each of them.
__device__ __forceinline__ uint32_t group_sum(uint32_t v, int lanes) {
  for (int d = 1; d < lanes; d <<= 1) v += __shfl_xor(v, d);
  return v;
}
__device__ __forceinline__ uint64_t inclusive_sum(uint64_t v) {
  const int lane = threadIdx.x & 63;
  for (int d = 1; d < 64; d <<= 1) {
    const uint64_t o = __shfl_up(v, d);
    v += lane >= d ? o : 0ull;
  }
  return v;
}

// Where every tier segment of the arena starts, where an item's kept positions do, and the rows of every tier: the plan that
// the host makes for the chunk table when it has the counts (pack_impl), here for the packing kernels, so that they wait for
// no table.  One workgroup; 2^k lanes add up an item's counts, and the items are a prefix sum apart.
__device__ __forceinline__ void plan_part(const ScatterArgs& a) {
  __shared__ uint64_t s_sum[2][4];
  const PlanArgs& p = a.plan;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int lanes = 64;                          // per item
  while (lanes > 1 && static_cast<int64_t>(lanes) * p.n_items > 256) lanes >>= 1;
  const int per_round = 256 / lanes, sub = tid & (lanes - 1);
  uint64_t units0 = 0, kept0 = 0;          // of the earlier rounds' items
  for (int i0 = 0; i0 < p.n_items; i0 += per_round) {
    const int item = i0 + tid / lanes;
    const bool in = item < p.n_items;
    const ItemOf it(a.batch, in ? item : 0);
    const int nb = in ? (it.T + kPartBlock - 1) / kPartBlock : 0, first = it.blk0;
    uint32_t cnt[4] = {0, 0, 0, 0};
#pragma unroll 4
    for (int b = sub; b < nb; b += lanes) {
      const int4 c = block_counts(a.blk_counts, first + b);
      cnt[0] += c.x; cnt[1] += c.y; cnt[2] += c.z; cnt[3] += c.w;
    }
    uint32_t words = 0, steps = 0;         // channel-wise: 32-bit words of a K row, its quantized steps
    if (p.bits_ch) {
      // Channels of every tier, eight bits each (at most 128).  Widths are one bit each; of a map that holds others, which the host
      // refuses, the sums mean nothing.  Four pieces' loads before the first sum: one after the other, a word at a time, they made the
      // launch 12.0 us for 88 items and 7.0 for 32; now 4.7 and 5.2, what it takes for a few.  (All eight pieces of a map, which one lane
      // has where there are more than 128 items, took 163 registers, a wavefront per SIMD from every workgroup of the launch: 128
      // token-wise items of 20K tokens 9.6 -> 12.5 us, eight of 128K 6.0 -> 7.4.)
      uint32_t ch = 0;
      constexpr int kPieces = kHeadDim / 16, kAtOnce = 4;
      const Bytes16* map = reinterpret_cast<const Bytes16*>(p.bits_ch + static_cast<int64_t>(in ? item : 0) * kHeadDim);
#pragma unroll 1
      for (int k0 = 0; k0 * lanes < kPieces; k0 += kAtOnce) {
        Bytes16 v[kAtOnce];
#pragma unroll
        for (int k = 0; k < kAtOnce; ++k) {
          const int piece = sub + (k0 + k) * lanes;
          v[k] = Bytes16{{0, 0, 0, 0}};
          if (in && piece < kPieces) v[k] = map[piece];
        }
#pragma unroll
        for (int k = 0; k < kAtOnce; ++k)
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int t = 0; t < 4; ++t) ch += static_cast<uint32_t>(__popc(v[k].v[e] & (0x10101010u >> t))) << (8 * t);
      }
      ch = group_sum(ch, lanes);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t slots = k_tier_slots(k, (ch >> (8 * k)) & 0xFF);
        words += slots * (16 >> k) / 32;
        if (k > 0) steps += slots / 4;
      }
      words = (words + 1) & ~1u;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) cnt[k] = group_sum(cnt[k], lanes);
    SegmentUnits size[4];
    uint64_t units = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      size[k] = segment_units(k, cnt[k], p.bits_ch != nullptr, static_cast<int>(words), static_cast<int>(steps), p.per_unit != 0);
      units += (size[k].k_data + size[k].k_meta) + (size[k].v_data + size[k].v_meta);
    }
    const uint32_t kept = cnt[0] + cnt[1] + cnt[2] + cnt[3];
    const uint64_t own_u = in && sub == 0 ? units : 0ull, own_k = in && sub == 0 ? kept : 0ull;
    const uint64_t inc_u = inclusive_sum(own_u), inc_k = inclusive_sum(own_k);
    __syncthreads();                       // (the sums of the round before are used up)
    if (lane == 63) {
      s_sum[0][wave] = inc_u;
      s_sum[1][wave] = inc_k;
    }
    __syncthreads();
    uint64_t u = units0 + inc_u - own_u, at = kept0 + inc_k - own_k;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      if (w < wave) { u += s_sum[0][w]; at += s_sum[1][w]; }
      units0 += s_sum[0][w];
      kept0 += s_sum[1][w];
    }
    if (in && sub == 0) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        p.counts[item * 4 + k] = static_cast<int32_t>(cnt[k]);
        p.idx_base[item * 4 + k] = static_cast<int64_t>(at);
        at += cnt[k];
        const uint64_t own[4] = {size[k].k_data, size[k].k_meta, size[k].v_data, size[k].v_meta};
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          p.seg_off[(static_cast<int64_t>(item) * 4 + k) * 4 + g] = static_cast<int64_t>(u * kSegAlign);
          u += own[g];
        }
      }
    }
  }
}

// Row layout of an item's channel-wise K tiles (make_item_k is the host's) by the first wavefront: two channels per lane.
__device__ __forceinline__ void layout_part(const PlanArgs& p, int item) {
  const int lane = threadIdx.x;
  ItemK* out = p.items_k + item;
  int tier[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) tier[h] = tier_slot(p.bits_ch[static_cast<int64_t>(item) * kHeadDim + 64 * h + lane]);
  const uint64_t below = (1ull << lane) - 1ull;
  uint32_t slot = 0, words = 0, steps = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint64_t lo = __ballot(tier[0] == k), hi = __ballot(tier[1] == k);
    const uint32_t n_lo = __popcll(lo), n = n_lo + __popcll(hi), slots = k_tier_slots(k, n);
    if (tier[0] == k) out->slot_ch[slot + __popcll(lo & below)] = static_cast<int16_t>(lane);
    if (tier[1] == k) out->slot_ch[slot + n_lo + __popcll(hi & below)] = static_cast<int16_t>(64 + lane);
    if (lane < slots - n) out->slot_ch[slot + n + lane] = -1;
    words += slots * (16 >> k) / 32;
    if (lane == 0) {
      out->slot_base[k] = static_cast<int16_t>(slot);
      out->word_end[k] = static_cast<int16_t>(words);
      if (k == 0) out->n_steps16 = static_cast<int16_t>(slots / 4);
    }
    if (k > 0) steps += slots / 4;
    slot += slots;
  }
  for (int j = slot + lane; j < kMaxSlots; j += 64) out->slot_ch[j] = -1;
  if (lane == 0) {
    out->n_slots = static_cast<int16_t>(slot);
    out->n_words = static_cast<int16_t>(words);
    out->n_words_padded = static_cast<int16_t>((words + 1) & ~1u);
    out->n_qsteps = static_cast<int16_t>(steps);
    out->kt_bytes = k_tile_bytes(static_cast<int>((words + 1) & ~1u));
    out->km_bytes = k_meta_bytes(static_cast<int>(steps));
  }
}

__global__ __launch_bounds__(256) void tier_scatter_kernel(ScatterArgs a) {
  static_assert(kPartBlock == 1024, "256 threads of four tokens");
  static_assert(kCopyThreads == 256, "copies in workgroups of this kernel");
  __shared__ int s_before[4][4], s_all[4][4];
  __shared__ uint64_t s_wave[4];
  if (static_cast<int>(blockIdx.x) < a.extra) {
    const int b = static_cast<int>(blockIdx.y) * a.extra + static_cast<int>(blockIdx.x), copies = a.copy.first[a.copy.n];
    if (b == 0) plan_part(a);
    else if (b <= copies) copy_part(a.copy, b - 1);
    return;
  }
  const int item = blockIdx.y, block = static_cast<int>(blockIdx.x) - a.extra;
  const ItemOf it(a.batch, item);
  const int T = it.T;
  const int t0 = block * kPartBlock;
  if (t0 >= T) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t tok_off = it.off;
  const uint8_t* b = a.bits + tok_off + t0;
  const int n = min(kPartBlock, T - t0), u = 4 * tid;
  uint32_t four = 0;                       // tokens past the end: evicted
  if (u + 3 < n) four = reinterpret_cast<const Bytes4*>(b + u)->v;
  else
    for (int e = 0; e < 4; ++e)
      if (u + e < n) four |= static_cast<uint32_t>(b[u + e]) << (8 * e);
  int before[4] = {0, 0, 0, 0}, all[4] = {0, 0, 0, 0};      // kept tokens of the item's earlier blocks, of all of them
  const int n_blocks = (T + kPartBlock - 1) / kPartBlock;
  for (int i = tid; i < n_blocks; i += 256) {
    const int4 x = block_counts(a.blk_counts, it.blk0 + i);
    const int c[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      all[k] += c[k];
      before[k] += i < block ? c[k] : 0;
    }
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int sum = static_cast<int>(wave_scan(static_cast<uint32_t>(before[k])));
    const int total = static_cast<int>(wave_scan(static_cast<uint32_t>(all[k])));
    if (lane == 63) {
      s_before[wave][k] = sum;
      s_all[wave][k] = total;
    }
  }
  int slot[4];
  uint64_t mine = 0;                       // this thread's tokens per tier, 16 bits each
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    slot[e] = tier_slot(static_cast<uint8_t>(four >> (8 * e)));
    mine += slot[e] >= 0 ? 1ull << (16 * slot[e]) : 0ull;
  }
  const uint64_t incl = static_cast<uint64_t>(wave_scan(static_cast<uint32_t>(mine))) |
                        static_cast<uint64_t>(wave_scan(static_cast<uint32_t>(mine >> 32))) << 32;   // (at most 256 each)
  if (lane == 63) s_wave[wave] = incl;
  __syncthreads();
  if (wave == 0 && block == 0 && a.plan.bits_ch) layout_part(a.plan, item);
  uint64_t rank = incl - mine;
  for (int w = 0; w < wave; ++w) rank += s_wave[w];
  int first[4], higher = 0;                // first of the block in its tier's list
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    first[k] = higher + s_before[0][k] + s_before[1][k] + s_before[2][k] + s_before[3][k];
    higher += s_all[0][k] + s_all[1][k] + s_all[2][k] + s_all[3][k];
  }
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (slot[e] >= 0) {
      const int k = slot[e];
      const int base = k == 0 ? first[0] : k == 1 ? first[1] : k == 2 ? first[2] : first[3];
      const int at = base + static_cast<int>((rank >> (16 * k)) & 0xFFFF);
      if (at < T) a.tier_idx[tok_off + at] = t0 + u + e;      // (a map that will be refused has blocks that were not counted)
      rank += 1ull << (16 * k);
    }
}

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

struct PackArgs {
  const uint16_t* K;
  const uint16_t* V;
  const int32_t* tier_idx;     // scratch: an item's kept positions from its first token's place on, tier after tier
  int32_t* tier_idx_out;       // the same without gaps: a tier's from idx_base on
  const int64_t* idx_base;     // [items][4]
  const int32_t* counts;       // [items][4]
  const int64_t* seg_off;      // [items][4][4]
  uint8_t* arena;
  const ItemK* items_k;        // [items] (mixed mode)
  uint32_t* k_range;           // [items][128][2]: ordered-integer images of a channel's minimum and maximum over all
                               // retained tokens (one scale per channel, App. B), or null (groups of 32 tokens)
  int32_t row_wide;            // token rows: one scale and offset per row (App. B's per-token format), repeated in
                               // the row's four metadata slots, instead of one per group of 32 channels
  int32_t extra;               // leading workgroups of every grid row that copy
  CopyArgs copy;
  Batch batch;
};

// monotone map float -> uint32 (and back), so that integer atomic min / max order floats
__device__ __forceinline__ uint32_t float_to_ordered(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float ordered_to_float(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

// The tile of a workgroup: the tiles of an item stand in the order of its tiers, 16, 8, 4, 2 (blockIdx.x counts them).
struct TileOf {
  int ti, n, tile, before;     // tier, rows of the segment, tile inside the segment, rows of the higher tiers; ti = 4: past the item's last
  __device__ __forceinline__ TileOf(const PackArgs& a, int item, int b) : ti(4), n(0), tile(0), before(0) {
    const int4 c = reinterpret_cast<const int4*>(a.counts)[item];
    const int rows[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int t = (rows[k] + kTile64 - 1) / kTile64;
      if (ti == 4) {
        if (b < t) {
          ti = k; n = rows[k]; tile = b;
        } else {
          b -= t;
          before += rows[k];
        }
      }
    }
  }
};

// The quantizer of one group: scale, offset and codes.  The correctly rounded quotient d / s without the division
// sequence, by Markstein's scheme (IBM J. Res. Dev. 34, 1990): q0 = d * y with y the hardware reciprocal of s, remainder
// r = d - q0 s exact in one fused multiply-add, q = q0 + r y.  The reciprocal is within one unit in the last place, not
// correctly rounded as the theorem asks; tests/test_quotient.py finds the IEEE quotient all the same for every fp16 s and
// all three y, at 128 million numerators around the half-integers and of differences of bf16 numbers.  A group with a scale
// or offset that is not finite takes the division.
// The scale's division by the largest code Q goes the same way with the correctly rounded 1 / Q, which is the theorem's case.
struct Quant {
  float m, s, y;
  _Float16 sh, mh;
  bool finite;
  // Q: the largest code, inv_q: 1 / Q; EXACT: by division
  template <bool EXACT = false>
  __device__ __forceinline__ void set(float mn, float mx, float Q, float inv_q) {
    mn = mn + 0.0f;            // canonical +0
    const float range = mx - mn;
    float q;
    if constexpr (EXACT) {
      q = range / Q;
    } else {
      const float q0 = range * inv_q;
      q = __builtin_fmaf(__builtin_fmaf(-q0, Q, range), inv_q, q0);
      q = __builtin_copysignf(q, range);         // (-0 of a group of -0)
      asm("" : "+v"(q));       // rounded to fp32 before it is rounded to fp16 (else one instruction does both)
    }
    sh = static_cast<_Float16>(q);               // round to nearest even
    mh = static_cast<_Float16>(mn);
    s = static_cast<float>(sh);
    m = static_cast<float>(mh);
    finite = fabsf(s) < INFINITY && fabsf(m) < INFINITY;     // (false for NaN)
    y = s == 0.0f ? 0.0f : __builtin_amdgcn_rcpf(s);
  }
  // The code: the low 16 bits of what comes back (rounded to an integer by the addition of 1.5 x 2^23, whose low half is
  // zero; clamped before, which is the same as after).  EXACT: by division
  template <bool EXACT>
  __device__ __forceinline__ uint32_t code(float x, float Q) const {
    const float d = x - m;
    float q;
    if constexpr (EXACT) {
      q = d / s;
    } else {                   // (with a finite s = 0: y = 0, q = 0)
      const float q0 = d * y;
      q = __builtin_fmaf(__builtin_fmaf(-q0, s, d), y, q0);
    }
    const float t = fminf(fmaxf(q, 0.0f), Q);
    return __float_as_uint((EXACT && s == 0.0f ? 0.0f : t) + 12582912.0f);
  }
};
// two codes as the halves of a word; four as its bytes, one after the other
__device__ __forceinline__ uint32_t code_halves(uint32_t lo, uint32_t hi) { return __builtin_amdgcn_perm(hi, lo, 0x05040100u); }
template <int I>
__device__ __forceinline__ uint32_t code_byte(uint32_t word, uint32_t code) {      // code in byte I, zeros above it
  return __builtin_amdgcn_perm(code, word, I == 1 ? 0x0C0C0400u : I == 2 ? 0x0C040100u : 0x04020100u);
}

constexpr int kQuadXor1 = 0xB1, kQuadXor2 = 0x4E;

__device__ __forceinline__ void unpack8(const uint4& v, float (&x)[8]) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    x[2 * j] = bf16_lo(w[j]);
    x[2 * j + 1] = bf16_hi(w[j]);
  }
}

// Minimum and maximum over a quad of lanes, over rows of 16.  (A minimum that reads another lane is one instruction; out of
// fminf the compiler makes three, because it cannot tell that what comes from another lane is no signalling NaN.  Two wait
// states stand between a write to a register and its use by another lane.)
__device__ __forceinline__ void quad_range(float& mn, float& mx) {
  asm("s_nop 1\n\t"
      "v_min_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "v_max_f32_dpp %1, %1, %1 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 0\n\t"
      "v_min_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
      "v_max_f32_dpp %1, %1, %1 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf"
      : "+v"(mn), "+v"(mx));
}
__device__ __forceinline__ void row_range(float& mn, float& mx) {      // after quad_range
  asm("s_nop 1\n\t"
      "v_min_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
      "v_max_f32_dpp %1, %1, %1 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 0\n\t"
      "v_min_f32_dpp %0, %0, %0 row_mirror row_mask:0xf bank_mask:0xf\n\t"
      "v_max_f32_dpp %1, %1, %1 row_mirror row_mask:0xf bank_mask:0xf"
      : "+v"(mn), "+v"(mx));
}

// Quantizes the 8 channels this lane holds of a token row (the 16 lanes of a row hold it in order, four lanes a group of
// 32 channels); codes as Quant::code gives them.
template <int BITS, bool EXACT>
__device__ __forceinline__ void quantize_row(const uint4& raw, int row_wide, Quant& g, uint32_t (&c)[8]) {
  constexpr float kMost = static_cast<float>((1 << BITS) - 1), kInvMost = 1.0f / kMost;
  float x[8];
  unpack8(raw, x);
  float mn = fminf(fminf(fminf(x[0], x[1]), fminf(x[2], x[3])), fminf(fminf(x[4], x[5]), fminf(x[6], x[7])));
  float mx = fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])), fmaxf(fmaxf(x[4], x[5]), fmaxf(x[6], x[7])));
  quad_range(mn, mx);
  if (row_wide) row_range(mn, mx);
  g.set<EXACT>(mn, mx, kMost, kInvMost);
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    if constexpr (EXACT) __builtin_amdgcn_sched_barrier(0);      // (eight divisions side by side take 40 registers)
    c[j] = g.code<EXACT>(x[j], kMost);
  }
}

// Tiers 8/4/2: the layout the decode kernels' 4x4x4 MFMA steps want.  A wavefront lane owns a run of 4*BITS 32-bit words,
// word W of lane L stored at byte 1024*(W/4) + 16*L + 4*(W%4).  The run holds four groups of BITS words; a group is
// read in eight steps of four codes: with F = 16/BITS fields per 16-bit half, step s reads field s % F of both
// halves of the word pair s / F, i.e. code k of step s sits at word 2*(s/F) + k/2, bit 16*(k%2) + BITS*(s%F).
//   K: lane = token r; group = c / 32; c % 32 = 4*step + k        (a lane holds one token's row)
//   V: lane = 32*(r/32) + c % 32; group = c / 32; r % 32 = 4*step + k   (a lane holds one channel for 32 tokens)
// Metadata tile = 1024 bytes: K row-major per token [4 scales][4 offsets]; V per block of 4 tokens 4 groups x 16
// bytes: the group's scales of the 4 tokens, then its offsets.
// K words: this lane's two steps of its group; the lanes of a group OR their fields together.  dst: k_words_at of the row's
// tile, plus 16 bytes per row.
template <int BITS>
__device__ __forceinline__ int k_words_at(int grp, int p) {
  const int W = BITS * grp + (BITS == 8 ? 2 * p : BITS == 4 ? (p & 2) : 0);
  return 1024 * (W >> 2) + 4 * (W & 3);
}
template <int BITS>
__device__ __forceinline__ void store_k_words(const uint32_t (&c)[8], uint8_t* dst, int p) {
  const auto word = [&](int k) __attribute__((always_inline)) {     // codes k, k + 1 of steps 2 p and 2 p + 1
    return code_halves(c[k], c[k + 1]) | (code_halves(c[4 + k], c[5 + k]) << BITS);
  };
  uint2 w = make_uint2(word(0), word(2));
  if constexpr (BITS == 4) {               // fields 2 (p % 2), 2 (p % 2) + 1 of word pair p / 2
    const int sh = 8 * (p & 1);
    w.x <<= sh;
    w.y <<= sh;
    w.x |= dpp_u32<kQuadXor1>(w.x);
    w.y |= dpp_u32<kQuadXor1>(w.y);
  } else if constexpr (BITS == 2) {        // fields 2 p, 2 p + 1 of the group's only word pair
    const int sh = 4 * p;
    w.x <<= sh;
    w.y <<= sh;
    w.x |= dpp_u32<kQuadXor1>(w.x);
    w.y |= dpp_u32<kQuadXor1>(w.y);
    w.x |= dpp_u32<kQuadXor2>(w.x);
    w.y |= dpp_u32<kQuadXor2>(w.y);
  }
  if (BITS == 8 || (BITS == 4 && (p & 1) == 0) || (BITS == 2 && p == 0)) *reinterpret_cast<uint2*>(dst) = w;
}

// V codes go through LDS: s_vc[channel][token] bytes, 68 bytes per channel (four tokens of a channel are one word of a
// lane, and both the writes and the reads spread over the banks).
constexpr int kVcStride = 68;
template <int BITS>
__device__ __forceinline__ void store_v_words(const uint8_t* s_vc, uint8_t* tile) {
  constexpr int F = 16 / BITS;
  const int L = threadIdx.x & 63, G = threadIdx.x >> 6;    // lane of the layout, channel group
  const uint32_t* src = reinterpret_cast<const uint32_t*>(s_vc + (32 * G + (L & 31)) * kVcStride + 32 * (L >> 5));
  uint32_t w[BITS];
#pragma unroll
  for (int i = 0; i < BITS; ++i) w[i] = 0;
#pragma unroll
  for (int st = 0; st < 8; ++st) {         // the four tokens of a step: bytes 0, 1 -> halves of one word, 2, 3 -> the other
    const uint32_t d = src[st];
    w[2 * (st / F)] |= __builtin_amdgcn_perm(0u, d, 0x0C010C00u) << (BITS * (st % F));
    w[2 * (st / F) + 1] |= __builtin_amdgcn_perm(0u, d, 0x0C030C02u) << (BITS * (st % F));
  }
  if constexpr (BITS == 2) {
    *reinterpret_cast<uint2*>(tile + 1024 * (G >> 1) + 16 * L + 8 * (G & 1)) = make_uint2(w[0], w[1]);
  } else {
#pragma unroll
    for (int q = 0; q < BITS / 4; ++q)
      *reinterpret_cast<uint4*>(tile + 1024 * (G * (BITS / 4) + q) + 16 * L) =
          make_uint4(w[4 * q], w[4 * q + 1], w[4 * q + 2], w[4 * q + 3]);
  }
}

// One workgroup = one tile of 64 kept rows of any tier, K and V (V_ONLY: V, K of a channel-wise cache is packed by
// pack_k_group); rows past the segment's last are zero rows, so a tile is always written whole.  A wavefront gathers
// 16 rows, 16 lanes a row (whole 256-byte rows per load), a lane the same 8 channels of four consecutive tokens, which is
// what a step of the V layout takes; codes are made in registers and only V passes through LDS, as bytes.  Bound: HBM and
// plain ALUs (the gather: 0.94 GB at 5.3 TB/s, half reads of whole rows; 14 instructions per element).  128 items x 20K
// tokens, mostly 2- and 4-bit rows: 216 -> 172 us; a 128K-token layer 20.4 -> 16.6 us; V alone of 8 x 50K 17.3 -> 13.6.  Before,
// positions were loaded row by row, codes were converted one by one, and the division path, inlined beside every row, took the
// registers of a fifth workgroup.
constexpr int kTileLds = kTile64 * (kHeadDim + 8) * 2;
// (The kernels find the tile and the item: inside of this function and of pack_k_group, which the compiler simplifies by themselves first,
// the item's number went through vector registers and back: K of 8 x 50K tokens 24.8 -> 24.4 us, its V 14.65 -> 14.25.)
// item_row: the item's first token; s_buf: kTileLds bytes for V codes, or bf16 V rows of the 16-bit tier; s_km: K metadata
template <bool V_ONLY>
__device__ __forceinline__ void pack_tile(const PackArgs& a, int item, const TileOf& t, int64_t item_row, uint8_t* s_buf, uint16_t (*s_km)[8]) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane >> 4, c16 = lane & 15, grp = c16 >> 2, p = c16 & 3;
  const int row0 = 16 * wave + 4 * lr;     // this lane's rows row0 .. row0 + 3 of the tile
  const int valid = min(kTile64, t.n - t.tile * kTile64);
  const int32_t* idx = a.tier_idx + item_row + t.before + static_cast<int64_t>(t.tile) * kTile64;
  if (tid < valid) a.tier_idx_out[a.idx_base[item * 4 + t.ti] + static_cast<int64_t>(t.tile) * kTile64 + tid] = idx[tid];
  uint4 kq[4], vq[4];
  // All positions, then all rows, without a branch (with one per row every position was waited for behind the rows before
  // it: four round trips instead of two).  Rows past the segment's last repeat it and become zeros.
  const auto gather = [&](int first) __attribute__((always_inline)) {
    int pos[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) pos[i] = idx[min(first + i, valid - 1)];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t src = (item_row + pos[i]) * kHeadDim + c16 * 8;
      if constexpr (!V_ONLY) kq[i] = *reinterpret_cast<const uint4*>(a.K + src);
      vq[i] = *reinterpret_cast<const uint4*>(a.V + src);
    }
    if (valid < kTile64) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (first + i >= valid) {
          if constexpr (!V_ONLY) kq[i] = make_uint4(0, 0, 0, 0);
          vq[i] = make_uint4(0, 0, 0, 0);
        }
    }
  };
  gather(row0);
  const int64_t* so = a.seg_off + (static_cast<int64_t>(item) * 4 + t.ti) * 4;
  const int bits = 16 >> t.ti;
  uint8_t* kd = a.arena + so[0] + static_cast<int64_t>(t.tile) * (kTile64 * kHeadDim / 8) * bits;
  uint8_t* vd = a.arena + so[2] + static_cast<int64_t>(t.tile) * (kTile64 * kHeadDim / 8) * bits;
  if (t.ti == 0) {
    if constexpr (!V_ONLY) {               // bf16 rows, row-major
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        *reinterpret_cast<uint4*>(kd + (row0 + i) * (kHeadDim * 2) + c16 * 16) = kq[i];
        *reinterpret_cast<uint4*>(vd + (row0 + i) * (kHeadDim * 2) + c16 * 16) = vq[i];
      }
    } else {
      // 16-bit V rows with the lane assignment of the quantized V tiers: lane 32 (r / 32) + c % 32 holds channel c for
      // the 32 tokens of its tile half, eight tokens per 16-byte unit; unit u = 4 (c / 32) + (r % 32) / 8 sits at byte
      // 1024 u + 16 lane of the 16 KiB tile
      constexpr int kStride = kHeadDim + 8;
      uint16_t* s_rows = reinterpret_cast<uint16_t*>(s_buf);
#pragma unroll
      for (int i = 0; i < 4; ++i) *reinterpret_cast<uint4*>(s_rows + (row0 + i) * kStride + c16 * 8) = vq[i];
      __syncthreads();
      uint32_t* dst = reinterpret_cast<uint32_t*>(vd);
      for (int word = tid; word < kTile64 * kHeadDim / 2; word += 256) {
        const int u = word >> 8, l = (word >> 2) & 63, t8 = 2 * (word & 3);
        const int r = 32 * (l >> 5) + 8 * (u & 3) + t8, c = 32 * (u >> 2) + (l & 31);
        dst[word] = s_rows[r * kStride + c] | (static_cast<uint32_t>(s_rows[(r + 1) * kStride + c]) << 16);
      }
    }
    return;
  }
  uint8_t* km = a.arena + so[1] + static_cast<int64_t>(t.tile) * 1024;
  uint8_t* vm = a.arena + so[3] + static_cast<int64_t>(t.tile) * 1024;
  // this wavefront's rows; false: some group's scale or offset is not finite, and everything has to be done again by division
  const auto quantize = [&](auto bits_c, auto exact_c) __attribute__((always_inline)) {
    constexpr int BITS = decltype(bits_c)::value;
    constexpr bool kExact = decltype(exact_c)::value;
    uint64_t odd = 0;
    if constexpr (!V_ONLY) {
      uint8_t* kw = kd + k_words_at<BITS>(grp, p) + 16 * row0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        Quant g;
        uint32_t c[8];
        __builtin_amdgcn_sched_barrier(0);     // row by row: registers decide how many workgroups are resident
        quantize_row<BITS, kExact>(kq[i], a.row_wide, g, c);
        odd |= __builtin_amdgcn_ballot_w64(!g.finite);
        store_k_words<BITS>(c, kw + 16 * i, p);
        if (p == 0) {
          s_km[row0 + i][grp] = __builtin_bit_cast(unsigned short, g.sh);
          s_km[row0 + i][4 + grp] = __builtin_bit_cast(unsigned short, g.mh);
        }
      }
    }
    uint32_t sc[4], of[4], packed[8];      // packed: the four tokens' codes of a channel, one byte each
    const auto row = [&](auto ic) __attribute__((always_inline)) {
      constexpr int I = decltype(ic)::value;
      Quant g;
      uint32_t c[8];
      __builtin_amdgcn_sched_barrier(0);
      quantize_row<BITS, kExact>(vq[I], a.row_wide, g, c);
      odd |= __builtin_amdgcn_ballot_w64(!g.finite);
      sc[I] = __builtin_bit_cast(unsigned short, g.sh);
      of[I] = __builtin_bit_cast(unsigned short, g.mh);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        if constexpr (I == 0) packed[j] = c[j]; else packed[j] = code_byte<I>(packed[j], c[j]);
      }
    };
    row(std::integral_constant<int, 0>{});
    row(std::integral_constant<int, 1>{});
    row(std::integral_constant<int, 2>{});
    row(std::integral_constant<int, 3>{});
#pragma unroll
    for (int j = 0; j < 8; ++j) *reinterpret_cast<uint32_t*>(s_buf + (c16 * 8 + j) * kVcStride + row0) = packed[j];
    if (p == 0)                            // block row0 / 4 of the tile, group grp
      *reinterpret_cast<uint4*>(vm + 16 * row0 + 16 * grp) =
          make_uint4(sc[0] | (sc[1] << 16), sc[2] | (sc[3] << 16), of[0] | (of[1] << 16), of[2] | (of[3] << 16));
    return odd == 0;
  };
  const auto tile = [&](auto bits_c) __attribute__((always_inline)) {
    if (!quantize(bits_c, std::false_type{})) {
      int again = row0;
      asm("" : "+v"(again));               // (or the addresses would be kept for it)
      gather(again);
      quantize(bits_c, std::true_type{});
    }
    __syncthreads();
    store_v_words<decltype(bits_c)::value>(s_buf, vd);
  };
  if (t.ti == 1) tile(std::integral_constant<int, 8>{});
  else if (t.ti == 2) tile(std::integral_constant<int, 4>{});
  else tile(std::integral_constant<int, 2>{});
  if constexpr (!V_ONLY) {
    if (tid < kTile64) *reinterpret_cast<uint4*>(km + 16 * tid) = *reinterpret_cast<const uint4*>(&s_km[tid][0]);
  }
}

// the copies that ride along: the leading workgroups of every grid row
__device__ __forceinline__ bool copied_along(const PackArgs& a) {
  static_assert(kCopyThreads == 256, "copies in workgroups of these kernels");
  if (static_cast<int>(blockIdx.x) >= a.extra) return false;
  const int b = static_cast<int>(blockIdx.y) * a.extra + static_cast<int>(blockIdx.x);
  if (b < a.copy.first[a.copy.n]) copy_part(a.copy, b);
  return true;
}

template <bool V_ONLY>
__global__ __launch_bounds__(256, 5) void pack_tile_kernel(PackArgs a) {
  __shared__ __align__(16) uint8_t s_buf[kTileLds];
  __shared__ __align__(16) uint16_t s_km[V_ONLY ? 1 : kTile64][8];
  if (copied_along(a)) return;
  const int item = blockIdx.y;
  const TileOf t(a, item, static_cast<int>(blockIdx.x) - a.extra);
  if (t.ti == 4) return;
  pack_tile<V_ONLY>(a, item, t, ItemOf(a.batch, item).off, s_buf, s_km);
}

// ---- mixed mode -------------------------------------------------------------------------------------------------
// One scale per channel over all retained tokens (App. B): the channel's minimum and maximum over the kept rows of
// all four tiers of the item.  k_range starts at (0xFFFFFFFF, 0).
// Bound: HBM (the kept rows once).  A wavefront's load is four rows, 16 bytes per lane, and kRangeLoads of them are in flight
// with the positions of the next ones; the order of bf16 numbers is that of 16-bit integers, two to a register, as
// float_to_ordered maps them.  Few workgroups per item, because each ends in 256 atomics on the item's 256 words.
// 8 items of 50K tokens, seven in ten kept, 154 -> 17 us, 2 of 128K 351 -> 17, 128 of 64K 1380 -> 281 (5.3 TB/s); before, a lane
// loaded two bytes of one row at a time, each row behind its position.
constexpr int kRangeThreads = 512, kRangeLoads = 8, kRangeRows = kRangeThreads / 16 * kRangeLoads;
using ushort2v = __attribute__((ext_vector_type(2))) unsigned short;
using short2v = __attribute__((ext_vector_type(2))) short;
__global__ __launch_bounds__(kRangeThreads) void k_channel_range_kernel(PackArgs a) {
  constexpr int kParts = kRangeThreads / 16;
  __shared__ uint4 s_part[2][kParts][16];            // smallest, largest: [rows of a load][channels 8 c16 ..]
  const int item = blockIdx.y, tid = threadIdx.x, part = tid >> 4, c16 = tid & 15;
  const int4 n4 = reinterpret_cast<const int4*>(a.counts)[item];
  const int kept = n4.x + n4.y + n4.z + n4.w;
  const int row0 = blockIdx.x * kRangeRows, step = static_cast<int>(gridDim.x) * kRangeRows;
  if (row0 >= kept) return;                          // (the whole workgroup)
  const int64_t item_row = ItemOf(a.batch, item).off;
  const int32_t* idx = a.tier_idx + item_row;
  const uint16_t* rows = a.K + item_row * kHeadDim + c16 * 8;
  union Piece { uint4 q; ushort2v h[4]; };
  Piece mn, mx;
  mn.q = make_uint4(0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu);
  mx.q = make_uint4(0, 0, 0, 0);
  int pos[kRangeLoads];
  const auto positions = [&](int r0) __attribute__((always_inline)) {      // rows past the last repeat it
#pragma unroll
    for (int i = 0; i < kRangeLoads; ++i) pos[i] = idx[min(r0 + i * kParts + part, kept - 1)];
  };
  positions(row0);
  for (int r0 = row0; r0 < kept; r0 += step) {
    Piece v[kRangeLoads];
#pragma unroll
    for (int i = 0; i < kRangeLoads; ++i) v[i].q = *reinterpret_cast<const uint4*>(rows + static_cast<int64_t>(pos[i]) * kHeadDim);
    if (r0 + step < kept) positions(r0 + step);
#pragma unroll
    for (int i = 0; i < kRangeLoads; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const ushort2v u = v[i].h[j];
        const ushort2v sign = __builtin_bit_cast(ushort2v, __builtin_bit_cast(short2v, u) >> short2v{15, 15});
        const ushort2v k = u ^ (sign | ushort2v{0x8000, 0x8000});
        mn.h[j] = __builtin_elementwise_min(mn.h[j], k);
        mx.h[j] = __builtin_elementwise_max(mx.h[j], k);
      }
  }
  s_part[0][part][c16] = mn.q;
  s_part[1][part][c16] = mx.q;
  __syncthreads();
  if (tid < kHeadDim) {                              // two channels each of the smallest (64 threads) and of the largest
    const bool largest = tid >= kHeadDim / 2;
    const int pair = tid & (kHeadDim / 2 - 1);
    const ushort2v* p = reinterpret_cast<const ushort2v*>(&s_part[largest][0][0]) + pair;
    ushort2v k = p[0];
#pragma unroll
    for (int i = 1; i < kParts; ++i) {
      const ushort2v o = p[i * (kHeadDim / 2)];
      k = largest ? __builtin_elementwise_max(k, o) : __builtin_elementwise_min(k, o);
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const uint32_t k16 = k[e], k32 = k16 << 16 | (k16 & 0x8000u ? 0u : 0xFFFFu);      // float_to_ordered of the number
      uint32_t* dst = &a.k_range[(static_cast<int64_t>(item) * kHeadDim + 2 * pair + e) * 2];
      if (largest) atomicMax(dst + 1, k32); else atomicMin(dst, k32);
    }
  }
}

// Channel-wise K of one 64-token tile (Sec. 3.2 Stage 3 on the retained tokens): every channel is quantized at
// its own bit-width over each half of the tile (one group = 32 consecutive retained tokens of one channel) and the
// codes are written in sorted-channel order.  Token r of the tile owns n_words_padded 32-bit words: word W at byte
// 1024 (W / 4) + 16 r + 4 (W % 4), the last two words of a row whose word count is not a multiple of four at
// 1024 (n / 4) + 8 r + 4 (W % 2).  Inside a word, slot 4k + e of a b-bit tier sits at bit
// 16 (e % 2) + b (e / 2) + 2 b k; a 16-bit word holds its two slots in its halves.
// Metadata: per token group G and quantized step sq (4 slots) 4 fp16 scales then 4 fp16 offsets at fp16 index
// 8 (G n_qsteps + sq).
//
// One workgroup = one token group of a tile, one thread = one slot of a word: its channel's 32 values in registers, quantized,
// the codes packed F tokens to a register (F = 32 / b fields of a word).  The F lanes that hold a word's slots then exchange
// fields so that lane f ends with the word of token f: a transposition of F x F fields in log2 F steps within a row of 16 lanes.
// Every tier starts at a row of lanes.  The words are staged in LDS and leave in 16-byte pieces.  Bound: a workgroup's chain of
// steps (rows, codes, words) and instruction issue; 160K rows 40 -> 32 us (a word put together field by field, each a channel
// number and a code out of LDS; and one code path per width, of which a wavefront with slots of three tiers took all three) -> 30
// (codes without conversions, all positions loaded before the rows) -> 24 (both groups of a tile in a workgroup before: half as
// many to cover each other's chains; 8 % fewer vector instructions alone had changed nothing).
// what lane ^ J holds (J = 1, 2, 4, 8, inside a row of 16)
template <int J>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v) {
  if constexpr (J == 1) return dpp_u32<kQuadXor1>(v);
  else if constexpr (J == 2) return dpp_u32<kQuadXor2>(v);
  else if constexpr (J == 8) return dpp_u32<0x128>(v);                    // row_ror:8
  else {
    const int lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x104, 0xF, 0x5, false);   // row_shl:4 into banks 0, 2
    return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(lo, static_cast<int>(v), 0x114, 0xF, 0xA, false));   // row_shr:4
  }
}
// One step of the transposition: fields of B bits whose index differs in bit J swap places with lane ^ J.
template <int B, int J>
__device__ __forceinline__ uint32_t exchange_fields(uint32_t v, int f) {
  uint32_t keep = 0;                   // fields with bit J clear
#pragma unroll
  for (int i = 0; i < 32 / B; ++i) keep |= (i & J) ? 0u : ((1u << B) - 1u) << (B * i);
  const bool up = (f & J) != 0;
  const uint32_t m = up ? ~keep : keep;
  const uint32_t o = lane_xor<J>(v);
  const uint32_t moved = __builtin_amdgcn_alignbit(o, o, up ? J * B : 32 - J * B);     // rotate right
  return (v & m) | (moved & ~m);
}
template <int B>
__device__ __forceinline__ uint32_t transpose_fields(uint32_t v, int f) {
  if constexpr (B <= 2) v = exchange_fields<B, 8>(v, f);
  if constexpr (B <= 4) v = exchange_fields<B, 4>(v, f);
  if constexpr (B <= 8) v = exchange_fields<B, 2>(v, f);
  return exchange_fields<B, 1>(v, f);
}

constexpr int kKThreads = 192;         // the most lanes a token group has
struct KGroupLds {
  static constexpr int kRowStride = kHeadDim + 8;
  static constexpr int kRowBytes = kKTokenGroup * kRowStride * 2, kWordBytes = kKTokenGroup * kMaxKRowWords * 4;
  uint8_t buf[kRowBytes > kWordBytes ? kRowBytes : kWordBytes];      // bf16 rows, then the group's words
  uint16_t sc[kHeadDim], of[kHeadDim];
  ItemK ik;
};
__device__ __forceinline__ void pack_k_group(const PackArgs& a, int item, const TileOf& t, int64_t item_row, int G, KGroupLds& lds) {
  constexpr int kRows = kKTokenGroup, kRowStride = KGroupLds::kRowStride;
  static_assert(kTile64 == 2 * kRows, "two workgroups a tile");
  uint8_t* const s_buf = lds.buf;
  uint16_t* const s_sc = lds.sc;
  uint16_t* const s_of = lds.of;
  ItemK& s_ik = lds.ik;
  const int valid = min(kTile64, t.n - t.tile * kTile64), vg = min(max(valid - kRows * G, 0), kRows);     // rows of the tile, of the group
  const int tid = threadIdx.x;
  const int64_t* so = a.seg_off + (static_cast<int64_t>(item) * 4 + t.ti) * 4;
  uint16_t* s_rows = reinterpret_cast<uint16_t*>(s_buf);
  {
    const int32_t* idx = a.tier_idx + item_row + t.before + static_cast<int64_t>(t.tile) * kTile64;
    constexpr int kPieces = kRows * 16, kLoads = (kPieces + kKThreads - 1) / kKThreads;      // 16 bytes each
    uint4 v[kLoads];
    int pos[kLoads];                     // all positions, then all rows (rows past the segment's last repeat it and become zeros)
#pragma unroll
    for (int i = 0; i < kLoads; ++i) pos[i] = idx[min(kRows * G + ((i * kKThreads + tid) >> 4), valid - 1)];
#pragma unroll
    for (int i = 0; i < kLoads; ++i)
      v[i] = *reinterpret_cast<const uint4*>(a.K + (item_row + pos[i]) * kHeadDim + (tid & 15) * 8);
    for (int i = tid; i < static_cast<int>(sizeof(ItemK) / 4); i += kKThreads)
      reinterpret_cast<uint32_t*>(&s_ik)[i] = reinterpret_cast<const uint32_t*>(a.items_k + item)[i];
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const int p = i * kKThreads + tid;
      if (p < kPieces)
        *reinterpret_cast<uint4*>(s_rows + (p >> 4) * kRowStride + (p & 15) * 8) = (p >> 4) < vg ? v[i] : make_uint4(0, 0, 0, 0);
    }
  }
  __syncthreads();

  // slots: lanes of a token group = words of a tier times slots of a word, tier by tier from a row of 16 on
  const int nwp = s_ik.n_words_padded, full = nwp & ~3;
  int start[5];
  start[0] = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k)
    start[k + 1] = start[k] + (((s_ik.word_end[k] - (k > 0 ? s_ik.word_end[k - 1] : 0)) * (2 << k) + 15) & ~15);
  const int lanes = start[4];            // at most 192
  const bool active = tid < lanes;
  int tier = 0, local = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (tid >= start[k] && tid < start[k + 1]) {
      tier = k;
      local = tid - start[k];
    }
  const int per_word = 2 << tier, f = local & (per_word - 1);
  const int first_word = tier > 0 ? s_ik.word_end[tier - 1] : 0, W = first_word + (local >> (tier + 1));
  const bool writes = active && W < s_ik.word_end[tier];
  int c = -1;                            // the slot's channel
  if (writes) {
    // slot 4 k + e of a word sits at bit 16 (e % 2) + b (e / 2) + 2 b k: field (F / 2) (e % 2) + e / 2 + 2 k
    const int half = per_word >> 1, e = 2 * (f & 1) + f / half, k4 = (f & (half - 1)) >> 1;
    c = s_ik.slot_ch[s_ik.slot_base[tier] + (W - first_word) * per_word + (tier == 0 ? f : 4 * k4 + e)];
  }
  float x[kKTokenGroup];                 // the channel's values, then their codes
#pragma unroll
  for (int r = 0; r < kKTokenGroup; ++r) x[r] = 0.f;
  if (c >= 0) {
#pragma unroll
    for (int r = 0; r < kKTokenGroup; ++r) x[r] = __uint_as_float(static_cast<uint32_t>(s_rows[r * kRowStride + c]) << 16);
    if (tier > 0) {                      // one path for all widths: a wavefront holds slots of several tiers
      uint16_t sc = 0, of = 0;
      if (vg > 0) {
        const float most = static_cast<float>((1 << (16 >> tier)) - 1);
        const float inv_most = tier == 1 ? 1.0f / 255.0f : tier == 2 ? 1.0f / 15.0f : 1.0f / 3.0f;
        float mn, mx;
        if (a.k_range) {   // the range of the whole unit
          mn = ordered_to_float(a.k_range[(static_cast<int64_t>(item) * kHeadDim + c) * 2]);
          mx = ordered_to_float(a.k_range[(static_cast<int64_t>(item) * kHeadDim + c) * 2 + 1]);
        } else {
          mn = x[0];
          mx = x[0];
          if (vg == kKTokenGroup) {
#pragma unroll
            for (int r = 1; r < kKTokenGroup; ++r) {
              mn = fminf(mn, x[r]);
              mx = fmaxf(mx, x[r]);
            }
          } else {
#pragma unroll
            for (int r = 1; r < kKTokenGroup; ++r) {
              mn = r < vg ? fminf(mn, x[r]) : mn;
              mx = r < vg ? fmaxf(mx, x[r]) : mx;
            }
          }
        }
        Quant g;
        g.set(mn, mx, most, inv_most);
        if (g.finite) {
#pragma unroll
          for (int r = 0; r < kKTokenGroup; ++r) x[r] = __uint_as_float(g.code<false>(x[r], most));
        } else {
          g.set<true>(mn, mx, most, inv_most);
#pragma unroll
          for (int r = 0; r < kKTokenGroup; ++r) x[r] = __uint_as_float(g.code<true>(x[r], most));
        }
        if (vg < kKTokenGroup) {
#pragma unroll
          for (int r = 0; r < kKTokenGroup; ++r) x[r] = r < vg ? x[r] : 0.f;
        }
        sc = __builtin_bit_cast(unsigned short, g.sh);
        of = __builtin_bit_cast(unsigned short, g.mh);
      } else {
#pragma unroll
        for (int r = 0; r < kKTokenGroup; ++r) x[r] = 0.f;
      }
      s_sc[c] = sc;
      s_of[c] = of;
    }
  }
  uint32_t out[16];                      // words of tokens F q + f
  const auto pack = [&](auto bits_c) __attribute__((always_inline)) {
    constexpr int B = decltype(bits_c)::value, F = 32 / B;
#pragma unroll
    for (int q = 0; q < kKTokenGroup / F; ++q) {
      uint32_t v = 0;
      if constexpr (B == 16) {
        v = (__float_as_uint(x[2 * q]) >> 16) | (__float_as_uint(x[2 * q + 1]) & 0xFFFF0000u);
      } else {
        // codes F / 2 apart stand in the two halves of a word
#pragma unroll
        for (int i = 0; i < F / 2; ++i)
          v |= code_halves(__float_as_uint(x[q * F + i]), __float_as_uint(x[q * F + F / 2 + i])) << (B * i);
      }
      out[q] = transpose_fields<B>(v, f);
    }
  };
  if (active) {
    if (tier == 3) pack(std::integral_constant<int, 2>{});
    else if (tier == 2) pack(std::integral_constant<int, 4>{});
    else if (tier == 1) pack(std::integral_constant<int, 8>{});
    else pack(std::integral_constant<int, 16>{});
  }
  __syncthreads();                       // the rows are used up: their memory takes the words
  uint32_t* s_words = reinterpret_cast<uint32_t*>(s_buf);
  const auto word_at = [&](int w, int r) __attribute__((always_inline)) {
    return w < full ? 4 * kRows * (w >> 2) + 4 * r + (w & 3) : kRows * full + 2 * r + (w - full);
  };
  if (writes) {
    const auto put = [&](auto bits_c) __attribute__((always_inline)) {
      constexpr int F = 32 / decltype(bits_c)::value;
#pragma unroll
      for (int q = 0; q < kKTokenGroup / F; ++q) s_words[word_at(W, F * q + f)] = out[q];
    };
    if (tier == 3) put(std::integral_constant<int, 2>{});
    else if (tier == 2) put(std::integral_constant<int, 4>{});
    else if (tier == 1) put(std::integral_constant<int, 8>{});
    else put(std::integral_constant<int, 16>{});
  }
  if (nwp > s_ik.n_words && tid < kRows) s_words[word_at(s_ik.n_words, tid)] = 0;
  __syncthreads();
  uint4* dst = reinterpret_cast<uint4*>(a.arena + so[0] + static_cast<int64_t>(t.tile) * s_ik.kt_bytes);
  const int quads = kRows * (full >> 2);   // pieces of 16 bytes: a token's four words; behind them two tokens' last two
  for (int idx = tid; idx < quads; idx += kKThreads)
    dst[(idx / kRows) * kTile64 + kRows * G + idx % kRows] = reinterpret_cast<const uint4*>(s_words)[idx];
  if (nwp > full && tid < kRows / 2) dst[2 * quads + (kRows / 2) * G + tid] = reinterpret_cast<const uint4*>(s_words)[quads + tid];
  // metadata; the segment's last tile also clears the bytes up to the next segment's alignment
  const int nqs = s_ik.n_qsteps, n_tiles = (t.n + kTile64 - 1) / kTile64;
  const bool last = t.tile == n_tiles - 1;
  if (a.k_range) {   // one record for the whole segment, written by its first tile
    uint16_t* meta1 = reinterpret_cast<uint16_t*>(a.arena + so[1]);
    const int words = 8 * nqs, padded = (2 * words + kSegAlign - 1) / kSegAlign * (kSegAlign / 2);
    if (t.tile == 0 && G == 0)
      for (int idx = tid; idx < padded; idx += kKThreads) {
        uint16_t v = 0;
        if (idx < words) {
          const int c = s_ik.slot_ch[s_ik.slot_base[1] + 4 * (idx >> 3) + (idx & 3)];
          if (c >= 0) v = (idx >> 2) & 1 ? s_of[c] : s_sc[c];
        }
        meta1[idx] = v;
      }
    return;
  }
  uint16_t* meta = reinterpret_cast<uint16_t*>(a.arena + so[1] + static_cast<int64_t>(t.tile) * s_ik.km_bytes) + 8 * nqs * G;
  const int64_t end = static_cast<int64_t>(n_tiles) * s_ik.km_bytes;
  const int pad = last && G == 1 ? static_cast<int>((kSegAlign - end % kSegAlign) % kSegAlign) / 2 : 0;
  for (int idx = tid; idx < 8 * nqs + pad; idx += kKThreads) {
    uint16_t v = 0;
    if (idx < 8 * nqs) {
      const int c = s_ik.slot_ch[s_ik.slot_base[1] + 4 * (idx >> 3) + (idx & 3)];
      if (c >= 0) v = (idx >> 2) & 1 ? s_of[c] : s_sc[c];
    }
    meta[idx] = v;
  }
}

__global__ __launch_bounds__(kKThreads, 6) void pack_k_mixed_kernel(PackArgs a) {
  __shared__ __align__(16) KGroupLds s;
  const int item = blockIdx.y;
  const TileOf t(a, item, blockIdx.x >> 1);
  if (t.ti == 4) return;
  pack_k_group(a, item, t, ItemOf(a.batch, item).off, blockIdx.x & 1, s);
}

// K and V of a channel-wise cache in one launch: k_groups workgroups per item for K, of three wavefronts (the fourth leaves at
// once), the others for V.  A small cache saves a launch (launch_quant_pack says where); in a large one K pays for the registers
// and the LDS of the V tiles.
__global__ __launch_bounds__(256, 5) void pack_mixed_kernel(PackArgs a, int k_groups) {
  __shared__ __align__(16) union {
    uint8_t tile[kTileLds];
    KGroupLds k;
  } s;
  if (copied_along(a)) return;
  const int item = blockIdx.y, b = static_cast<int>(blockIdx.x) - a.extra;
  if (b < k_groups) {
    if (threadIdx.x >= kKThreads) return;
    const TileOf t(a, item, b >> 1);
    if (t.ti != 4) pack_k_group(a, item, t, ItemOf(a.batch, item).off, b & 1, s.k);
  } else {
    const TileOf t(a, item, b - k_groups);
    if (t.ti != 4) pack_tile<true>(a, item, t, ItemOf(a.batch, item).off, s.tile, nullptr);
  }
}

}  // namespace

hipError_t launch_tier_count(const uint8_t* bits, const Batch& batch, int32_t* blk_counts, int max_T, hipStream_t st) {
  const int max_blk = (max_T + kPartBlock - 1) / kPartBlock, n_items = batch.n_seqs * batch.hkv;
  if (n_items == 0 || max_blk == 0) return hipSuccess;
  hipLaunchKernelGGL(tier_count_kernel, dim3(max_blk, n_items), dim3(256), 0, st, bits, reinterpret_cast<int4*>(blk_counts), batch);
  return hipGetLastError();
}

// The position lists, the plan and what `copy` holds (planned; the counts on their way to the host where nobody has posted them, fills,
// or nothing), in one launch.
hipError_t launch_tier_scatter(const uint8_t* bits, const Batch& batch, const int32_t* blk_counts, int32_t* tier_idx,
                               const PlanArgs& plan, int max_T, const CopyArgs& copy, hipStream_t st) {
  const int max_blk = (max_T + kPartBlock - 1) / kPartBlock, others = copy.first[copy.n] + 1;
  const ScatterArgs a{bits, reinterpret_cast<const int4*>(blk_counts), tier_idx, (others + plan.n_items - 1) / plan.n_items, plan, copy, batch};
  hipLaunchKernelGGL(tier_scatter_kernel, dim3(max_blk + a.extra, plan.n_items), dim3(256), 0, st, a);
  return hipGetLastError();
}

// max_tiles: the most 64-row tiles any item has over its tiers (at least one); k_range must hold (0xFFFFFFFF, 0) pairs on entry.
// `copy` (planned) goes along.
hipError_t launch_quant_pack(const uint16_t* K, const uint16_t* V, const int32_t* tier_idx, int32_t* tier_idx_out,
                             const PlanArgs& plan, const Batch& batch, uint8_t* arena, int max_tiles,
                             uint32_t* k_range, int row_wide, const CopyArgs& copy, hipStream_t st) {
  const int n_items = plan.n_items, extra = (copy.first[copy.n] + n_items - 1) / n_items;
  const PackArgs a{K, V, tier_idx, tier_idx_out, plan.idx_base, plan.counts, plan.seg_off, arena, plan.items_k,
                   k_range, row_wide, extra, copy, batch};
  const dim3 with_copies(max_tiles + extra, n_items), block(256);
  if (plan.items_k == nullptr) {
    hipLaunchKernelGGL(pack_tile_kernel<false>, with_copies, block, 0, st, a);
    return hipGetLastError();
  }
  if (k_range) {
    // 512 workgroups fill the chip; 16 per item are left where there are many items, 128 at most where there are few
    const int parts = std::min(std::max(512 / n_items, 16), 128), most = (max_tiles * kTile64 + kRangeRows - 1) / kRangeRows;
    hipLaunchKernelGGL(k_channel_range_kernel, dim3(std::max(1, std::min(parts, most)), n_items), dim3(kRangeThreads), 0, st, a);
  }
  // One launch for K and V where they are few workgroups, the launch's own time counts and the slower workgroups do not: a whole pass
  // over 1.7K to 6.7K tokens of 2 to 24 items (up to 2400 workgroups) 71.4 -> 67.6, 72.4 -> 69.6, 87.9 -> 84.4 and 109.2 -> 105.7 us, of
  // 32 items of 4K (5800) 117.0 -> 116.7, of 8 items of 50K and 39K tokens (11K, 14K) 162.0 -> 166.1 and 173.2 -> 174.6, of 12 of 55K
  // 304 -> 326.
  constexpr int64_t kTogether = 4096;
  if (static_cast<int64_t>(3 * max_tiles) * n_items <= kTogether) {
    hipLaunchKernelGGL(pack_mixed_kernel, dim3(3 * max_tiles + extra, n_items), block, 0, st, a, 2 * max_tiles);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(pack_k_mixed_kernel, dim3(2 * max_tiles, n_items), dim3(kKThreads), 0, st, a);
  hipLaunchKernelGGL(pack_tile_kernel<true>, with_copies, block, 0, st, a);
  return hipGetLastError();
}

}  // namespace rdkv
