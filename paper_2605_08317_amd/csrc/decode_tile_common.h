// Device helpers shared by the tile decode kernels (token-wise and mixed mode): operand types, the subnormal-fp16
// unpack of packed codes, tile loads, and the stages both kernels run after the logits of a 64-token tile are
// known: online softmax, P V over a token-wise V tile, and the end-of-chunk merge of a workgroup's wavefronts.
//
// Lane roles (v_mfma_f32_4x4x4_16B_f16, sixteen independent 4x4x4 blocks, lane = 4 * block + x):
//   logits    lane (block b, x = head j) holds tokens 4b..4b+3 of the tile in its four result registers
//   P V       A = p * scale of lane (b, head j) for its tokens, broadcast from block a to blocks 0..7 and from
//             block 8 + a to blocks 8..15 (cbsz = 3);  B = V codes: lane = (token half, channel of the group),
//             4 tokens per step;  D: lane holds 4 heads of one channel, summed over its token half.
#pragma once
#include "decode_merge.h"
#include "rdkv_internal.h"
#include "wave_ops.h"

namespace rdkv {
namespace tile {

typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kTile = 64;   // tokens per tile
constexpr float kNegBig = -1.0e30f;
constexpr float kLogitScale = 1.4426950408889634f * 0.08838834764831845f;   // log2(e) / sqrt(128)

// Codes enter the matrix cores as fp16 subnormals: a 16-bit pattern with a zero exponent field and the code in
// mantissa bits [fb, fb + b) is the number code * 2^fb * 2^-24 exactly, so one AND per pair of codes is the whole
// conversion.  The query operand of the K product is pre-multiplied by 2^(kQExp - fb); on the V side the power of
// two goes into p (per lane) and the accumulators are rescaled once per chunk.
constexpr int kQExp = 4;                                   // keeps the scaled query clear of fp16 underflow
constexpr float kKUnit = 1.0f / static_cast<float>(1 << (24 - kQExp));   // K partial products come out times this
constexpr float kXScale = kLogitScale * static_cast<float>(1 << (24 - kQExp));

// The probabilities exp2(x - running maximum) are carried times 2^kPExp, so that after the multiplication by a
// V scale they stay in fp16's normal range for flat attention over tens of thousands of tokens (p ~ 1e-5); the
// factor is returned by reporting the running maximum kPExp lower to the merge.  2^kPExp * scale must stay below
// 65504, which holds for V scales below 1023.
constexpr float kPExp = 6.0f;

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

typedef short short4v __attribute__((ext_vector_type(4)));
typedef uint32_t uint2v __attribute__((ext_vector_type(2)));

// four bf16 of an operand from two 32-bit words (a bit cast: a union of the two types is left in scratch memory)
__device__ __forceinline__ short4v bf4(uint32_t lo, uint32_t hi) { return __builtin_bit_cast(short4v, uint2v{lo, hi}); }

// the probabilities of a lane's four tokens as two truncated bf16 terms (the remainder of the first is exact in fp32)
__device__ __forceinline__ void split_bf16(const float (&p)[4], short4v& hi, short4v& lo) {
  uint32_t hb[4], lb[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    hb[i] = __float_as_uint(p[i]) & 0xFFFF0000u;
    lb[i] = __float_as_uint(p[i] - __uint_as_float(hb[i]));
  }
  hi = bf4((hb[0] >> 16) | hb[1], (hb[2] >> 16) | hb[3]);
  lo = bf4((lb[0] >> 16) | (lb[1] & 0xFFFF0000u), (lb[2] >> 16) | (lb[3] & 0xFFFF0000u));
}

union Pack4 {
  half4 h;
  half2v p[2];
  uint32_t u[2];
};

// value held by lane i of this lane's quad
template <int I>
__device__ __forceinline__ uint32_t quad_bcast(uint32_t v) { return dpp_u32<I * 0x55>(v); }

template <int G>
struct GroupIndex {
  static constexpr int value = G;
};

// Query on the A side of the K products: lane (block b, head j) holds channels 8 b .. 8 b + 7 of head 4 hs + j, that is
// the operands of steps 2 b and 2 b + 1, and a product broadcasts the block that holds its step (cbsz = 4).  Sixteen
// bytes per lane are the whole query of four heads, loaded by each wavefront for itself: no LDS, no barrier before the
// first tile.  (With the query on the B side every lane needed every step's operand, 32 eight-byte LDS reads per tile and
// head set: 1100 cycles of LDS bandwidth for eight wavefronts.)
__device__ __forceinline__ uint4 load_query(const uint16_t* __restrict__ q, int head, int g, int blk) {
  return head < g ? *reinterpret_cast<const uint4*>(q + head * kHeadDim + 8 * blk) : make_uint4(0, 0, 0, 0);
}

// The K products leave lane = token with the four heads of a set in its registers; the softmax and P V want lane (block,
// head) with the block's four tokens: a 4x4 transposition inside each quad of lanes, in two steps that exchange registers
// with lane ^ 1 and lane ^ 2.  Moves only, so that a head whose logits are not finite stays by itself: products with unit
// vectors, which turn the block as well, spread its NaN over the set (0 x NaN).
// Two forms.  Written plainly it becomes eight moves and eight selections, which the compiler spreads over the code around.
// A selection that takes one side from another lane is one instruction: half as many, in one piece (FEW).  That is better
// where the vector issue is full, with two head sets over token rows (16 ragged sequences with 8 query heads 44.1 us with
// the products, 44.3 plainly, 44.1 so), and worse elsewhere (one channel-wise 64K sequence, 4 query heads 16.9, 16.2, 17.1; a
// batch of 16, 8 query heads, 32K tokens 97.1, 97.5, 99.0).
// (A selection of that kind reads its mask, the lanes that keep their own register, from vcc.  Two wait states stand between
// a write to a register and its use by another lane.)
#define RDKV_TURN_MASK(M_) "s_mov_b32 vcc_lo, " #M_ "\n\ts_mov_b32 vcc_hi, " #M_ "\n\t"
#define RDKV_TURN_1(D_, OTHER_, OWN_) "v_cndmask_b32_dpp " D_ ", " OTHER_ ", " OWN_ ", vcc quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
#define RDKV_TURN_2(D_, OTHER_, OWN_) "v_cndmask_b32_dpp " D_ ", " OTHER_ ", " OWN_ ", vcc quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
template <int HS, bool FEW>
__device__ __forceinline__ void to_head_lanes(const float (&xt)[HS][4], int j, float (&x)[HS][4]) {
  const bool odd = (j & 1) != 0, high = (j & 2) != 0;
#pragma unroll
  for (int hs = 0; hs < HS; ++hs) {
    float t[4];
    if constexpr (FEW) {
#pragma unroll
      for (int i = 0; i < 4; ++i) x[hs][i] = xt[hs][i];
      asm("s_nop 1\n\t"
          RDKV_TURN_MASK(0x55555555) RDKV_TURN_1("%4", "%1", "%0") RDKV_TURN_1("%6", "%3", "%2")
          RDKV_TURN_MASK(0xaaaaaaaa) RDKV_TURN_1("%5", "%0", "%1") RDKV_TURN_1("%7", "%2", "%3")
          RDKV_TURN_MASK(0x33333333) RDKV_TURN_2("%0", "%6", "%4") RDKV_TURN_2("%1", "%7", "%5")
          RDKV_TURN_MASK(0xcccccccc) RDKV_TURN_2("%2", "%4", "%6") RDKV_TURN_2("%3", "%5", "%7")
          : "+v"(x[hs][0]), "+v"(x[hs][1]), "+v"(x[hs][2]), "+v"(x[hs][3]), "=&v"(t[0]), "=&v"(t[1]), "=&v"(t[2]), "=&v"(t[3])
          :
          : "vcc");
    } else {
#pragma unroll
      for (int k = 0; k < 4; k += 2) {
        const float from1 = dpp_f32<0xB1>(xt[hs][k + 1]), from0 = dpp_f32<0xB1>(xt[hs][k]);   // quad_perm [1, 0, 3, 2]
        t[k] = odd ? from1 : xt[hs][k];
        t[k + 1] = odd ? xt[hs][k + 1] : from0;
      }
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const float from2 = dpp_f32<0x4E>(t[k + 2]), from0 = dpp_f32<0x4E>(t[k]);             // quad_perm [2, 3, 0, 1]
        x[hs][k] = high ? from2 : t[k];
        x[hs][k + 2] = high ? t[k + 2] : from0;
      }
    }
  }
}
#undef RDKV_TURN_2
#undef RDKV_TURN_1
#undef RDKV_TURN_MASK

// Field position of step s inside a 16-bit half, which right-shifted copy of the word it is read from, and the bit
// offset that remains after that shift (the code then reads as code * 2^fb * 2^-24).
template <int TIER>
struct Step {
  static constexpr int F = 16 / TIER;                                     // fields per half
  __host__ __device__ static constexpr int pair(int s) { return s / F; }
  __host__ __device__ static constexpr int field(int s) { return s % F; }
  __host__ __device__ static constexpr int copy(int s) {
    return TIER == 8 ? 0 : TIER == 4 ? field(s) / 2 : field(s) / 3;
  }
  __host__ __device__ static constexpr int fb(int s) {
    return TIER == 8 ? 0 : TIER == 4 ? 4 * (field(s) % 2) : 2 * (field(s) % 3);
  }
  static constexpr int kCopies = TIER == 8 ? 1 : TIER == 4 ? 2 : 3;
  static constexpr int kShift = TIER == 4 ? 8 : 6;                        // right shift between copies
};

// The 4 codes of step s of a group whose words are gw[0..TIER): two words, fp16 subnormals in both halves.
template <int TIER>
__device__ __forceinline__ half4 step_operand(const uint32_t (&gw)[Step<TIER>::kCopies][TIER], int s) {
  using S = Step<TIER>;
  Pack4 r;
  const int p = S::pair(s);
  if constexpr (TIER == 8) {
    // byte f of each half, zero-extended: both selections go through the byte permute (mixing it with a plain
    // AND of the same register was seen to be scheduled with the AND done in place before the permute read it)
    const uint32_t sel = S::field(s) ? 0x0C030C01u : 0x0C020C00u;
    r.u[0] = __builtin_amdgcn_perm(0u, gw[0][2 * p], sel);
    r.u[1] = __builtin_amdgcn_perm(0u, gw[0][2 * p + 1], sel);
  } else {
    const uint32_t mask = (TIER == 4 ? 0x000F000Fu : 0x00030003u) << S::fb(s);
    r.u[0] = gw[S::copy(s)][2 * p] & mask;
    r.u[1] = gw[S::copy(s)][2 * p + 1] & mask;
  }
  return r.h;
}

template <int TIER>
__device__ __forceinline__ void group_words(const uint4 (&raw)[TIER], int grp, uint32_t (&gw)[Step<TIER>::kCopies][TIER]) {
  using S = Step<TIER>;
#pragma unroll
  for (int w = 0; w < TIER; ++w) {
    const int W = grp * TIER + w;
    const uint4 c = raw[W >> 2];
    const uint32_t v = (W & 3) == 0 ? c.x : (W & 3) == 1 ? c.y : (W & 3) == 2 ? c.z : c.w;
    gw[0][w] = v;
#pragma unroll
    for (int k = 1; k < S::kCopies; ++k) gw[k][w] = v >> (k * S::kShift);
  }
}

template <int TIER>
__device__ __forceinline__ void load_tile_side(uint4 (&raw)[TIER], const uint8_t* __restrict__ data, int tile, int lane) {
  const uint8_t* p = data + static_cast<int64_t>(tile) * (kTile * 16 * TIER) + lane * 16;
#pragma unroll
  for (int i = 0; i < TIER; ++i) raw[i] = *reinterpret_cast<const uint4*>(p + i * 1024);
}

// sixteen bytes of a buffer (a type the host's compiler does not know), zeros past its end
template <class Buffer>
__device__ __forceinline__ uint4 load_uint4(Buffer buf, int at) {
  const auto v = __builtin_amdgcn_raw_buffer_load_b128(buf, at, 0, 0);
  return make_uint4(v[0], v[1], v[2], v[3]);
}

__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Running state of one wavefront over its tiles of a chunk: per head set the running maximum and sum of the
// online softmax (lanes of head j; the sum carries this lane's factor kappa), the output accumulators
// acc[hs][grp][i] (head 4 hs + i, channel 32 grp + lane % 32, summed over this lane's token half), and the offset
// sums offv[hs][i] = kappa * sum_t p m of head 4 hs + i and channel group lane % 4 over the tokens of this lane's block.
template <int HS>
struct Run {
  float m[HS], l[HS];
  floatx4 acc[HS][4];
  floatx4 offv[HS];
  __device__ __forceinline__ void init() {
#pragma unroll
    for (int hs = 0; hs < HS; ++hs) {
      m[hs] = kNegBig;
      l[hs] = 0.f;
      offv[hs] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int grp = 0; grp < 4; ++grp) acc[hs][grp] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
  }
};

// Padded rows of a chunk's last tile take no part in the softmax.
template <int HS>
__device__ __forceinline__ void mask_rows(float (&x)[HS][4], int tile, int rows, int blk) {
  if ((tile + 1) * kTile > rows) {
#pragma unroll
    for (int hs = 0; hs < HS; ++hs)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (tile * kTile + 4 * blk + i >= rows) x[hs][i] = -INFINITY;
  }
}

// Online softmax per head over the logits x (in units of 1 / kXScale) of a tile; probabilities carried times
// 2^(kPExp + lk): lk = log2 of the lane's factor kappa on the V side (0 where there is none), which the exponential
// applies for free; the running sum carries the same factor and finish_chunk takes it out again.
// The reference is the running maximum itself: the token that sets it has p = 2^kPExp, exact in fp16 as is its product with an
// fp16 V scale, and that is the token with the most weight.  (A reference that stays until a logit exceeds it by 2^5 saved 0 to
// 3 % and rounded that token like any other: mean error with logits of a spread of 4 powers of two 2.0e-4 -> 3.5e-4, of 9
// 0.6e-4 -> 2.2e-4.)  The lanes are asked for their maximum only where one of them has exceeded it: 16 ragged sequences with 8
// query heads per KV head 42.1 -> 41.7 us, 8 layers of 4K tokens 58.5 -> 58.0, with 4 heads or fewer the same.
template <int HS>
__device__ __forceinline__ void softmax_tile(const float (&x)[HS][4], Run<HS>& run, float (&p)[HS][4], float lk = 0.f) {
#pragma unroll
  for (int hs = 0; hs < HS; ++hs) {
    const float most = max_of_four(x[hs][0], x[hs][1], x[hs][2], x[hs][3]);
    if (__any(most > run.m[hs])) {
      const float m_new = fmaxf(run.m[hs], head_max(most));
      const float alpha = fast_exp2((run.m[hs] - m_new) * kXScale);
      run.l[hs] *= alpha;
      const uint32_t au = __builtin_bit_cast(uint32_t, alpha);
      const float ah[4] = {__builtin_bit_cast(float, quad_bcast<0>(au)), __builtin_bit_cast(float, quad_bcast<1>(au)),
                           __builtin_bit_cast(float, quad_bcast<2>(au)), __builtin_bit_cast(float, quad_bcast<3>(au))};
#pragma unroll
      for (int i = 0; i < 4; ++i) {   // row i of the accumulators is head i
#pragma unroll
        for (int grp = 0; grp < 4; ++grp) run.acc[hs][grp][i] *= ah[i];
        run.offv[hs][i] *= ah[i];
      }
      run.m[hs] = m_new;
    }
    const float neg_mc = (kPExp + lk) - run.m[hs] * kXScale;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      p[hs][i] = fast_exp2(__builtin_fmaf(x[hs][i], kXScale, neg_mc));
      run.l[hs] += p[hs][i];
    }
  }
}

// log2 of kappa = 2^-fb of the field this lane's block is read from on the V side (block a = blk % 8 feeds step a)
template <int TIER>
__device__ __forceinline__ float v_log2_kappa(int blk) {
  float lk = 0.0f;
#pragma unroll
  for (int a = 0; a < 8; ++a)
    if ((blk & 7) == a) lk = -static_cast<float>(Step<TIER>::fb(a));
  return lk;
}

// P V over a token-wise V tile of tier TIER (8, 4, 2).  fill_gw(GroupIndex<G>, gw) delivers the code words of
// channel group G (and their shifted copies); vmeta = group (lane % 4)'s scales (x, y) and offsets (z, w) of
// tokens 4 blk + 0..3; p = the probabilities times the lane's kappa (softmax_tile with lk).
// The offsets go through one more product: A = p (4 heads x the block's 4 tokens), B = this lane's offsets (4 tokens
// of channel group lane % 4), so that lane (block, j) gathers sum_t p m of the four heads for group j -- with the
// same rounded p that multiplies the codes, which keeps the two halves of sum_t p (s code + m) consistent.
template <int TIER, int HS, class FillGw>
__device__ __forceinline__ void pv_tile_groups(FillGw&& fill_gw, const uint4& vmeta, const float (&p)[HS][4],
                                               Run<HS>& run) {
  using S = Step<TIER>;
  Pack4 ph[HS], ob;
  ob.u[0] = vmeta.z;
  ob.u[1] = vmeta.w;
#pragma unroll
  for (int hs = 0; hs < HS; ++hs) {
    ph[hs].p[0] = half2v{static_cast<_Float16>(p[hs][0]), static_cast<_Float16>(p[hs][1])};
    ph[hs].p[1] = half2v{static_cast<_Float16>(p[hs][2]), static_cast<_Float16>(p[hs][3])};
    run.offv[hs] = __builtin_amdgcn_mfma_f32_4x4x4f16(ph[hs].h, ob.h, run.offv[hs], 0, 0, 0);
  }
#define RDKV_PV_GROUP(G_)                                                                                      \
  {                                                                                                            \
    __builtin_amdgcn_sched_barrier(0);                                                                         \
    /* V scales of tokens 4 blk + 0..3: lane G_ of the quad holds group G_'s (x, y) */                         \
    Pack4 sv, pa[HS];                                                                                          \
    sv.u[0] = quad_bcast<G_>(vmeta.x); sv.u[1] = quad_bcast<G_>(vmeta.y);                                      \
    _Pragma("unroll") for (int hs = 0; hs < HS; ++hs) {                                                        \
      pa[hs].p[0] = ph[hs].p[0] * sv.p[0];                                                                     \
      pa[hs].p[1] = ph[hs].p[1] * sv.p[1];                                                                     \
    }                                                                                                          \
    uint32_t gw[S::kCopies][TIER];                                                                             \
    fill_gw(GroupIndex<G_>{}, gw);                                                                             \
    RDKV_PV_STEP(G_, 0) RDKV_PV_STEP(G_, 1) RDKV_PV_STEP(G_, 2) RDKV_PV_STEP(G_, 3)                            \
    RDKV_PV_STEP(G_, 4) RDKV_PV_STEP(G_, 5) RDKV_PV_STEP(G_, 6) RDKV_PV_STEP(G_, 7)                            \
  }
#define RDKV_PV_STEP(G_, A_)                                                                                   \
  {                                                                                                            \
    const half4 b = step_operand<TIER>(gw, A_);                                                                \
    _Pragma("unroll") for (int hs = 0; hs < HS; ++hs)                                                          \
        run.acc[hs][G_] = __builtin_amdgcn_mfma_f32_4x4x4f16(pa[hs].h, b, run.acc[hs][G_], 3, A_, 0);          \
  }
  RDKV_PV_GROUP(0) RDKV_PV_GROUP(1) RDKV_PV_GROUP(2) RDKV_PV_GROUP(3)
#undef RDKV_PV_STEP
#undef RDKV_PV_GROUP
}

// the same with the whole tile's code words in registers
template <int TIER, int HS>
__device__ __forceinline__ void pv_tile(const uint4 (&vraw)[TIER], const uint4& vmeta, const float (&p)[HS][4],
                                        Run<HS>& run) {
  pv_tile_groups<TIER, HS>(
      [&](auto gi, uint32_t (&gw)[Step<TIER>::kCopies][TIER]) __attribute__((always_inline)) {
        group_words<TIER>(vraw, decltype(gi)::value, gw);
      },
      vmeta, p, run);
}

// Where a chunk's partial result goes and what the merge of its item needs.
struct ChunkOut {
  int item, slot, slot0, nslots;   // the chunk's item and partial slot; the item's first slot and slot count
};

// Floats of LDS the end of a chunk needs behind s_ml for the wavefronts' sums (launches that count: later the merge's).
__host__ __device__ constexpr int finish_lds_floats(int waves, int g) {
  return waves * g * kHeadDim > merge::merge_lds_floats(waves * 64) ? waves * g * kHeadDim : merge::merge_lds_floats(waves * 64);
}
// Floats of s_ml: per wavefront, head and channel group the maximum, the sum, the group's offset sum and a free word.
__host__ __device__ constexpr int ml_lds_floats(int waves, int hs) { return waves * hs * 4 * kGroupsPerRow * 4; }
template <int HS>
__device__ __forceinline__ constexpr int ml_at(int wave, int head, int group) {
  return ((wave * HS * 4 + head) * kGroupsPerRow + group) * 4;
}

// A wavefront is through with its tiles: the merging wavefronts of its heads start to look at whole partials.  The state words
// (decode_merge.h) come back, lane by lane; nothing waits for them here.
template <bool LOOK, int NWV>
__device__ __forceinline__ uint32_t ends_soon(int g, const MergeArgs& ma, const ChunkOut& co) {
  uint32_t state = merge::kAbsent;
  if constexpr (LOOK) {
    const int block = merge::own_block<NWV>();
    if (block < g * merge::kBlocks && co.nslots > 1) state = merge::clear_state(ma, co.slot, block, merge::kEndsSoon);
  }
  return state;
}

// Last part of a chunk's end, after s_ml and s_acc ([NWV][g][128] unnormalised sums times 1 / acc_scale, offset sums not
// included, each relative to its wavefront's own maximum) are written: one barrier, then a wavefront per head weighs and adds
// the NWV wavefronts' values, two channels a lane.  The weights are made once, lane w of each row of lanes that of wavefront
// w (by every lane for itself they were eight exponentials and eight more reads of LDS).  An item of a single chunk is finished
// here; otherwise the partial result is stored, for the item's merging workgroups (LOOK) or announced (decode_merge.h).
template <int HS, int NWV, bool LOOK>
__device__ __forceinline__ void store_partial(float acc_scale, int g, const float* s_ml, float* s_acc, const MergeArgs& ma,
                                              const ChunkOut& co) {
  const int lane = threadIdx.x & 63, ch = 2 * lane;
  const bool single = co.nslots == 1;
  const int64_t qh0 = static_cast<int64_t>(co.item) * g;
  __syncthreads();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  constexpr int kHeads = (4 * HS + NWV - 1) / NWV;
#pragma unroll
  for (int k = 0; k < kHeads; ++k) {      // (in a loop that is one, the answer of ends_soon would be waited for in front of it)
    const int head = wave + k * NWV;
    if (head >= g) break;
    // row of lanes = channel group, which is that of the lane's two channels
    const float2 ml = *reinterpret_cast<const float2*>(s_ml + ml_at<HS>(lane & (NWV - 1), head, lane >> 4));
    float2 a[NWV];
    float off[NWV];      // (added wavefront by wavefront: the two terms of an output nearly cancel)
#pragma unroll
    for (int w = 0; w < NWV; ++w) {
      a[w] = *reinterpret_cast<const float2*>(s_acc + (w * g + head) * kHeadDim + ch);
      off[w] = s_ml[ml_at<HS>(w, head, lane >> 4) + 2];
    }
    const float mm = row_max(ml.x);
    const float f = fast_exp2(ml.x - mm);
    const bool own = (lane & 15) < NWV;      // (the other lanes repeat one)
    const float l = row_sum(own ? ml.y * f : 0.f);
    float v0 = 0.f, v1 = 0.f;
#pragma unroll
    for (int w = 0; w < NWV; ++w) {
      const float fw = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(f), w));
      v0 = __builtin_fmaf(__builtin_fmaf(a[w].x, acc_scale, off[w]), fw, v0);
      v1 = __builtin_fmaf(__builtin_fmaf(a[w].y, acc_scale, off[w]), fw, v1);
    }
    if (single) {
      float* o = ma.out + (qh0 + head) * kHeadDim + ch;
      o[0] = l > 0.f ? v0 / l : 0.f;
      o[1] = l > 0.f ? v1 / l : 0.f;
      if (lane == 0 && ma.lse != nullptr) ma.lse[qh0 + head] = l > 0.f ? (mm + __log2f(l)) * 0.6931471805599453f : -INFINITY;
    } else if constexpr (LOOK) {
      float* rec = merge::look_record(ma, co.slot, head, ch >> 4);
      merge::store_agent2(rec + (ch & 15), merge::present(v0), merge::present(v1));
      if ((ch & 15) == 0) merge::store_agent2(rec + 16, merge::present(mm), merge::present(l));
    } else {
      merge::store_agent2(ma.part_acc + (static_cast<int64_t>(co.slot) * g + head) * kHeadDim + ch, v0, v1);
      if (lane == 0) merge::store_agent2(ma.part_ml + (static_cast<int64_t>(co.slot) * g + head) * 2, mm, l);
    }
  }
  if constexpr (!LOOK) {
    if (single) return;
    merge::partial_stores_done();
    __syncthreads();     // every partial store has landed, and nobody reads s_ml / s_acc any more
    merge::arrive_and_merge<NWV * 64, 4 * HS>(ma, co.item, co.slot0, co.nslots, g, s_acc);
  }
}

// End of a chunk: take the lane's factor kappa = 2^lk out of the running sums, add the token halves of the accumulators and
// the blocks' offset sums, and merge the workgroup's NWV wavefronts through LDS (store_partial; acc_scale = 2^24 where the V
// codes entered as fp16 subnormals).
// s_ml: ml_lds_floats(NWV, HS); s_acc: finish_lds_floats(NWV, g) floats.  ALIAS: the two areas overlap LDS that
// the tile loop used, so a barrier separates the two uses.
template <int HS, bool ALIAS, int NWV, bool LOOK>
__device__ __forceinline__ uint32_t finish_chunk(Run<HS>& run, float acc_scale, float lk, int g, float* s_ml,
                                                 float* s_acc, const MergeArgs& ma, const ChunkOut& co) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const float inv_kappa = __builtin_ldexpf(1.0f, static_cast<int>(-lk));   // lk is a small integer
  const uint32_t state = ends_soon<LOOK, NWV>(g, ma, co);
  if constexpr (ALIAS) __syncthreads();
#pragma unroll
  for (int hs = 0; hs < HS; ++hs) {
    run.l[hs] = head_sum(run.l[hs] * inv_kappa);
    // lanes (block, j) hold head i's sum_t p m of channel group j over the block's tokens.  The sums over the blocks, the
    // four heads turned into the four rows of lanes on the way
    float o[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = run.offv[hs][i] * inv_kappa;
    swap_rows(o[0], o[1]);
    swap_rows(o[2], o[3]);
    float lo = o[0] + o[1], hi = o[2] + o[3];
    swap_halves(lo, hi);
    float off = lo + hi;
    off += dpp_f32<0x124>(off);
    off += dpp_f32<0x128>(off);
    if (lane < 16)        // (block, j) -> group block of head j; log2 domain from here on
      *reinterpret_cast<float2*>(s_ml + ml_at<HS>(wave, 4 * hs + (lane & 3), lane >> 2)) =
          make_float2(run.m[hs] * kXScale - kPExp, run.l[hs]);
    if ((lane & 12) == 0) s_ml[ml_at<HS>(wave, 4 * hs + (lane >> 4), lane & 3) + 2] = off;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int head = 4 * hs + i;
      const float v0 = halves_sum(run.acc[hs][0][i], run.acc[hs][1][i]), v1 = halves_sum(run.acc[hs][2][i], run.acc[hs][3][i]);
      if (head < g) {
        s_acc[(wave * g + head) * kHeadDim + lane] = v0;
        s_acc[(wave * g + head) * kHeadDim + 64 + lane] = v1;
      }
    }
  }
  store_partial<HS, NWV, LOOK>(acc_scale, g, s_ml, s_acc, ma, co);
  return state;
}

// A chunk of appended tokens (Sec. 3.3 Zone C: bf16 rows kept after the compression pass) on the same instruction
// and lane roles.  The tail is stored in 64-token tiles written by the append kernel: K tile = 16 KiB, word W (two
// bf16 channels 2W, 2W+1) of token r at byte 1024 (W / 4) + 16 r + 4 (W % 4), so a lane (= token) reads its row
// with sixteen coalesced 16-byte loads; V tile = 16 KiB in the layout of the 16-bit V tiles of mixed mode (lane
// 32 (r / 32) + c % 32 holds channel c, eight tokens per 16-byte unit u = 4 (c / 32) + (r % 32) / 8 at 1024 u).
template <int HS, bool ALIAS, int NWV, bool LOOK>
__device__ __forceinline__ uint32_t process_tail_tiles(const uint8_t* __restrict__ kd, const uint8_t* __restrict__ vd,
                                                   int rows, int g, const uint16_t* __restrict__ q,
                                                   float* s_ml, float* s_acc, const MergeArgs& ma,
                                                   const ChunkOut& co) {
  constexpr int kWaves = NWV;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int blk = lane >> 2, j = lane & 3;
  const int ntiles = (rows + kTile - 1) / kTile;
  constexpr int kTileBytes = kTile * kHeadDim * 2;
  uint4 qa[HS];      // raw bf16: the products are exact
#pragma unroll
  for (int hs = 0; hs < HS; ++hs) qa[hs] = load_query(q, 4 * hs + j, g, blk);
  Run<HS> run;
  run.init();
  const floatx4 zero4 = {0.f, 0.f, 0.f, 0.f};
  for (int tile = wave; tile < ntiles; tile += kWaves) {
    const uint8_t* kp = kd + static_cast<int64_t>(tile) * kTileBytes + 16 * lane;
    const uint8_t* vp = vd + static_cast<int64_t>(tile) * kTileBytes + 16 * lane;
    uint4 kq[16], vq[3][4];   // the K row and the first channel group of V in one round trip
#pragma unroll
    for (int i = 0; i < 16; ++i) kq[i] = *reinterpret_cast<const uint4*>(kp + 1024 * i);
#pragma unroll
    for (int i = 0; i < 4; ++i) vq[0][i] = *reinterpret_cast<const uint4*>(vp + 1024 * i);
    floatx4 a16[HS];
#pragma unroll
    for (int hs = 0; hs < HS; ++hs) a16[hs] = zero4;
    // step s = channels 4 s .. 4 s + 3 = words 2 s, 2 s + 1
#define RDKV_TAIL_K(I_)                                                                                         \
  _Pragma("unroll") for (int hs = 0; hs < HS; ++hs) {                                                          \
    a16[hs] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(bf4(qa[hs].x, qa[hs].y), bf4(kq[I_].x, kq[I_].y), a16[hs], 4, I_, 0); \
    a16[hs] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(bf4(qa[hs].z, qa[hs].w), bf4(kq[I_].z, kq[I_].w), a16[hs], 4, I_, 0); \
  }
    RDKV_TAIL_K(0) RDKV_TAIL_K(1) RDKV_TAIL_K(2) RDKV_TAIL_K(3) RDKV_TAIL_K(4) RDKV_TAIL_K(5) RDKV_TAIL_K(6)
    RDKV_TAIL_K(7) RDKV_TAIL_K(8) RDKV_TAIL_K(9) RDKV_TAIL_K(10) RDKV_TAIL_K(11) RDKV_TAIL_K(12) RDKV_TAIL_K(13)
    RDKV_TAIL_K(14) RDKV_TAIL_K(15)
#undef RDKV_TAIL_K
    __builtin_amdgcn_sched_barrier(0);   // the K registers are free: the other three channel groups of V
#pragma unroll
    for (int i = 0; i < 4; ++i) vq[1][i] = *reinterpret_cast<const uint4*>(vp + 1024 * (4 + i));
#pragma unroll
    for (int i = 0; i < 4; ++i) vq[2][i] = *reinterpret_cast<const uint4*>(vp + 1024 * (8 + i));
    float xt[HS][4], x[HS][4];
#pragma unroll
    for (int hs = 0; hs < HS; ++hs)
#pragma unroll
      for (int i = 0; i < 4; ++i) xt[hs][i] = a16[hs][i] * kKUnit;
    to_head_lanes<HS, HS == 2>(xt, j, x);
    mask_rows<HS>(x, tile, rows, blk);
    float p[HS][4];
    softmax_tile<HS>(x, run, p);
    short4v phi[HS], plo[HS];
#pragma unroll
    for (int hs = 0; hs < HS; ++hs) split_bf16(p[hs], phi[hs], plo[hs]);
    // P V: step a of a channel group = tokens 4a..4a+3 of this lane's token half (rows past the end are zero in the
    // tile and carry p = 0)
#define RDKV_TAIL_STEP(G_, A_, X_, Y_)                                                                          \
  {                                                                                                            \
    const short4v b = bf4(X_, Y_);                                                                             \
    _Pragma("unroll") for (int hs = 0; hs < HS; ++hs) {                                                        \
      run.acc[hs][G_] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(phi[hs], b, run.acc[hs][G_], 3, A_, 0);         \
      run.acc[hs][G_] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(plo[hs], b, run.acc[hs][G_], 3, A_, 0);         \
    }                                                                                                          \
  }
#define RDKV_TAIL_GROUP(G_, V_)                                                                                \
  RDKV_TAIL_STEP(G_, 0, V_[0].x, V_[0].y) RDKV_TAIL_STEP(G_, 1, V_[0].z, V_[0].w)                              \
  RDKV_TAIL_STEP(G_, 2, V_[1].x, V_[1].y) RDKV_TAIL_STEP(G_, 3, V_[1].z, V_[1].w)                              \
  RDKV_TAIL_STEP(G_, 4, V_[2].x, V_[2].y) RDKV_TAIL_STEP(G_, 5, V_[2].z, V_[2].w)                              \
  RDKV_TAIL_STEP(G_, 6, V_[3].x, V_[3].y) RDKV_TAIL_STEP(G_, 7, V_[3].z, V_[3].w)
    RDKV_TAIL_GROUP(0, vq[0])
#pragma unroll
    for (int i = 0; i < 4; ++i) vq[0][i] = *reinterpret_cast<const uint4*>(vp + 1024 * (12 + i));   // group 3
    RDKV_TAIL_GROUP(1, vq[1])
    RDKV_TAIL_GROUP(2, vq[2])
    RDKV_TAIL_GROUP(3, vq[0])
#undef RDKV_TAIL_GROUP
#undef RDKV_TAIL_STEP
  }
  return finish_chunk<HS, ALIAS, NWV, LOOK>(run, 1.0f, 0.f, g, s_ml, s_acc, ma, co);
}

}  // namespace tile
}  // namespace rdkv
