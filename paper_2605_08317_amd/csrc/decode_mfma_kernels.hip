// Split-K flash-decode over the quantized tiers (8/4/2 bit) of a token-wise cache (Sec. 3.3, Eq. 7) on the
// gfx950 matrix cores.
//
// With grouped-query attention the query heads of a KV head share every K/V byte.  The products run on
// v_mfma_f32_4x4x4_16B_f16: sixteen independent 4x4x4 blocks per instruction, four query heads on one side, so
// that no lane of the result is padding (a 16-wide head dimension would be three quarters empty at g = 4 and
// the plain ALUs, which apply the scales and the softmax to every result lane, are the scarce unit).
//
//   q K^T   A = the query, 4 heads x 4 channels: block b of the lanes holds steps 2b and 2b + 1, broadcast to all blocks
//           (cbsz = 4);  B = K codes: lane = token (64 per tile), 4 channels per step;  D: lane = token, four heads.
//           Eight steps cover a quantization group of 32 channels; the group's scale, the lane's own, multiplies the
//           partial product (fusion identity of App. B) and the offsets go through one more product with the group
//           sums of q.  Exchanges inside the quads then turn each block, so that lane (block b, head j) holds tokens
//           4b..4b+3.  With the query on the B side instead the result needed no turning, but every operand of it came
//           from LDS and every scale through four cross-lane moves: 16 ragged sequences with 8 query heads per KV head
//           45.4 -> 44.1 us, a layer of 16 MB 11.0 -> 10.7 us.
//   P V     A = p * scale of lane (b, head j) for its tokens 4b..4b+3, broadcast from block a to blocks 0..7 and
//           from block 8 + a to blocks 8..15 (cbsz = 3);  B = V codes: lane = (token half, channel of the group),
//           4 tokens per step;  D: lane holds 4 heads of one channel, summed over its token half.  One instruction
//           per (group, a): the V scale of a (token, group) is applied on the A side.
//
// Codes enter as fp16 subnormals: a 16-bit pattern with a zero exponent field and the code in mantissa bits
// [fb, fb + b) is the number code * 2^fb * 2^-24 exactly, so one AND per pair of codes is the whole conversion.
// The tile layout puts the four codes of a step in the two halves of two words at one field position; the
// power of two of the field is folded into the query operand (K side) or into p (V side, per lane).
// Everything a tile needs is loaded straight into registers in its final form; LDS holds only the merge of the wavefronts
// of a workgroup.
#include "decode_rows.h"

namespace rdkv {

namespace {

using namespace tile;

// One piece of a workgroup's work: `rows` rows of one tier of one item, NWV wavefronts interleaving over its tiles.
// The running softmax state `run` carries over from piece to piece (a workgroup may go through several tiers of its
// item); the sums that carry the lane's factor kappa of this tier take it on entry and give it back on exit.
// ROOMY: for launches of at most one workgroup per compute unit, where a wavefront may use twice the registers: K and V of
// an 8-bit tile are then in flight together.
template <int TIER, int HS, int NWV, bool ROOMY>
__device__ __forceinline__ void process_tiles(const uint8_t* __restrict__ kd, const uint8_t* __restrict__ km,
                                              const uint8_t* __restrict__ vd, const uint8_t* __restrict__ vm,
                                              int rows, int g, const uint16_t* __restrict__ q, Run<HS>& run) {
  constexpr int kWaves = NWV;
  using S = Step<TIER>;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int blk = lane >> 2, j = lane & 3;

  const int ntiles = (rows + kTile - 1) / kTile;

  // The query first: loads return in order, and its operands are made while the first tiles are on their way.
  uint4 qraw[HS];
#pragma unroll
  for (int hs = 0; hs < HS; ++hs) qraw[hs] = load_query(q, 4 * hs + j, g, blk);

  // ---- first tile's loads, issued before anything waits ------------------------------------------------
  // K and V of a tile sit in separate registers and are refilled each right after its last use, so a wavefront always has
  // its next tile in flight; of the 2-bit tiles (6 KiB) two.  Where registers are short, the K and V codes of an 8-bit tile
  // (18 KiB) take turns in one register set, and the other wavefronts of the SIMD cover the wait.
  constexpr bool kShare = TIER == 8 && !ROOMY;
  constexpr int kDepth = (TIER == 2 && HS == 1) ? 2 : 1;
  struct Regs {
    uint4 k[TIER], v[kShare ? 1 : TIER], kmeta, vmeta;
  };
  Regs regs[kDepth];
  // The V scales and offsets ahead of the V codes or behind them: P V needs the scales with the first codes, and loads return in
  // order.  Ahead: 32 layers of 128K tokens, 4 query heads per KV head, 299 -> 277 us, 8 of 32K 70.7 -> 69.3.  With two head sets it
  // is behind them: 8 layers of 4K tokens 58.0 us against 61.1 ahead, of 16K 75.0 and 79.5, of 32K 73.6 and 77.1 (the compiler
  // then waits for the V codes load by load in more places), 32K at 4 bits 136.7 and 135.0.  Launches of more workgroups than
  // compute units: the same either way.
  constexpr bool kMetaFirst = ROOMY && HS == 1;
  auto load_vmeta = [&](Regs& r, int t) __attribute__((always_inline)) {
    // lane (block, j) fetches group j's scales and offsets of tokens 4 blk + 0..3; the quad shares them below
    r.vmeta = *reinterpret_cast<const uint4*>(vm + static_cast<int64_t>(t) * 1024 + lane * 16);
  };
  auto load_k = [&](Regs& r, int t) __attribute__((always_inline)) {
    load_tile_side<TIER>(r.k, kd, t, lane);
    r.kmeta = *reinterpret_cast<const uint4*>(km + static_cast<int64_t>(t) * 1024 + lane * 16);
  };
  auto load_v = [&](Regs& r, int t) __attribute__((always_inline)) {
    if constexpr (kMetaFirst) load_vmeta(r, t);
    if constexpr (kShare) load_tile_side<TIER>(r.k, vd, t, lane); else load_tile_side<TIER>(r.v, vd, t, lane);
    if constexpr (!kMetaFirst) load_vmeta(r, t);
  };
#pragma unroll
  for (int dd = 0; dd < kDepth; ++dd) {
    regs[dd].kmeta = regs[dd].vmeta = make_uint4(0, 0, 0, 0);
    if (wave + dd * kWaves < ntiles) {
      load_k(regs[dd], wave + dd * kWaves);
      if constexpr (!kShare) load_v(regs[dd], wave + dd * kWaves);
    }
  }

  // ---- query operands (once per piece: the field positions folded into them depend on the tier) ----------------------
  // qop[hs][e]: q * 2^(kQExp - fb(step)) of step 2 blk + e; qhi, qlo: the sums of q over the four channel groups (k = group)
  // as two fp16 terms, for the K offsets.  A group's channels sit in one row of 16 lanes.
  half4 qop[HS][2], qhi[HS], qlo[HS];
#pragma unroll
  for (int hs = 0; hs < HS; ++hs) {
    const uint32_t w[4] = {qraw[hs].x, qraw[hs].y, qraw[hs].z, qraw[hs].w};
    float psum = 0.f;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      int fb = 0;      // of step st = 2 (blk % 4) + e of the group
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if ((blk & 3) == k) fb = S::fb(2 * k + e);
      const float f = ldexpf(1.0f, kQExp - fb);
      const float v0 = __uint_as_float(w[2 * e] << 16), v1 = __uint_as_float(w[2 * e] & 0xFFFF0000u);
      const float v2 = __uint_as_float(w[2 * e + 1] << 16), v3 = __uint_as_float(w[2 * e + 1] & 0xFFFF0000u);
      qop[hs][e] = half4{static_cast<_Float16>(v0 * f), static_cast<_Float16>(v1 * f), static_cast<_Float16>(v2 * f),
                         static_cast<_Float16>(v3 * f)};
      psum += (v0 + v1) + (v2 + v3);
    }
    psum += dpp_f32<0x124>(psum);
    psum += dpp_f32<0x128>(psum);
    float s0 = psum, s1 = psum;      // rows 0 .. 3 of 16 lanes = groups 0 .. 3: every lane gets all four
    swap_rows(s0, s1);
    float s2 = s0, s3 = s1;
    swap_halves(s0, s2);
    swap_halves(s1, s3);
    const float sg[4] = {s0, s1, s2, s3};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      qhi[hs][k] = static_cast<_Float16>(sg[k]);
      qlo[hs][k] = static_cast<_Float16>(sg[k] - static_cast<float>(qhi[hs][k]));
    }
  }

  const float lk = v_log2_kappa<TIER>(blk);
  {
    const float kappa = __builtin_ldexpf(1.0f, static_cast<int>(lk));
#pragma unroll
    for (int hs = 0; hs < HS; ++hs) {
      run.l[hs] *= kappa;
#pragma unroll
      for (int i = 0; i < 4; ++i) run.offv[hs][i] *= kappa;
    }
  }
  const floatx4 zero4 = {0.f, 0.f, 0.f, 0.f};

  auto do_tile = [&](Regs& r, const int tile) __attribute__((always_inline)) {
    const int next = tile + kDepth * kWaves;
    const bool more = next < ntiles;
    const uint4& kmeta = r.kmeta;

    // ---- logits xt[hs][i] of this lane's token and head 4 hs + i, in units of kKUnit ---------------------------------
    float xt[HS][4], x[HS][4];
    {
      // offsets x group sums of q (B: this lane's own token, k = group)
      Pack4 boff;
      boff.u[0] = kmeta.z;
      boff.u[1] = kmeta.w;
#pragma unroll
      for (int hs = 0; hs < HS; ++hs) {
        floatx4 d = __builtin_amdgcn_mfma_f32_4x4x4f16(qhi[hs], boff.h, zero4, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_4x4x4f16(qlo[hs], boff.h, d, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) xt[hs][i] = d[i] * kKUnit;
      }
#define RDKV_K_STEP(G_, S_)                                                                                        \
  {                                                                                                               \
    const half4 b = step_operand<TIER>(gw, S_);                                                                   \
    _Pragma("unroll") for (int hs = 0; hs < HS; ++hs)                                                             \
        dg[hs] = __builtin_amdgcn_mfma_f32_4x4x4f16(qop[hs][(S_) & 1], b, dg[hs], 4, (G_) * 4 + (S_) / 2, 0);     \
  }
#define RDKV_K_GROUP(G_)                                                                                           \
  {                                                                                                               \
    __builtin_amdgcn_sched_barrier(0); /* keep a group's unpacked words next to their use (register pressure) */  \
    uint32_t gw[S::kCopies][TIER];                                                                                \
    group_words<TIER>(r.k, G_, gw);                                                                               \
    floatx4 dg[HS];                                                                                               \
    _Pragma("unroll") for (int hs = 0; hs < HS; ++hs) dg[hs] = zero4;                                             \
    RDKV_K_STEP(G_, 0) RDKV_K_STEP(G_, 1) RDKV_K_STEP(G_, 2) RDKV_K_STEP(G_, 3)                                   \
    RDKV_K_STEP(G_, 4) RDKV_K_STEP(G_, 5) RDKV_K_STEP(G_, 6) RDKV_K_STEP(G_, 7)                                   \
    /* the token's scale of group G_: half G_ of (x, y) */                                                        \
    const float sf = static_cast<float>(__builtin_bit_cast(half2v, (G_) < 2 ? kmeta.x : kmeta.y)[(G_) & 1]);      \
    _Pragma("unroll") for (int hs = 0; hs < HS; ++hs)                                                             \
      _Pragma("unroll") for (int i = 0; i < 4; ++i) xt[hs][i] = __builtin_fmaf(sf, dg[hs][i], xt[hs][i]);         \
  }
      RDKV_K_GROUP(0) RDKV_K_GROUP(1) RDKV_K_GROUP(2) RDKV_K_GROUP(3)
#undef RDKV_K_GROUP
#undef RDKV_K_STEP
    }
    if constexpr (kShare) load_v(r, tile);   // the K codes are used up: their registers take this tile's V codes
    else if (more) load_k(r, next);          // K registers are free again

    to_head_lanes<HS, HS == 2>(xt, j, x);
    mask_rows<HS>(x, tile, rows, blk);
    float p[HS][4];
    softmax_tile<HS>(x, run, p, lk);
    if constexpr (kShare) pv_tile<TIER, HS>(r.k, r.vmeta, p, run); else pv_tile<TIER, HS>(r.v, r.vmeta, p, run);
    if (more) {               // V registers are free again
      if constexpr (kShare) load_k(r, next); else load_v(r, next);
    }
  };
  for (int tile = wave; tile < ntiles; tile += kDepth * kWaves) {
#pragma unroll
    for (int dd = 0; dd < kDepth; ++dd)
      if (tile + dd * kWaves < ntiles) do_tile(regs[dd], tile + dd * kWaves);
  }

  {   // the piece is done: the lane's factor leaves the sums again
    const float inv_kappa = __builtin_ldexpf(1.0f, static_cast<int>(-lk));
#pragma unroll
    for (int hs = 0; hs < HS; ++hs) {
      run.l[hs] *= inv_kappa;
#pragma unroll
      for (int i = 0; i < 4; ++i) run.offv[hs][i] *= inv_kappa;
    }
  }
}

// MULTI: workgroups may go through several tiers of their item (Chunk::next); without it every chunk is one tier and
// the tier's body ends in its own copy of the chunk's end, which saves a latency-bound launch 0.3 us.
template <int HS, int NWV, bool MULTI, bool ROOMY, bool LOOK>
__global__ __launch_bounds__(NWV * 64, ROOMY ? 2 : HS == 1 ? 4 : 3) void decode_tiles_kernel(
    const Chunk* __restrict__ chunks, const uint8_t* __restrict__ arena, const uint16_t* __restrict__ q,
    const int32_t* __restrict__ tail_len, int first, int g, MergeArgs ma) {
  extern __shared__ __align__(16) uint8_t smem[];
  Chunk ch = chunks[first + blockIdx.x];
  const int n_tail = *tail_len;      // with the chunk, not after it
  const uint16_t* qp = q + static_cast<int64_t>(ch.item) * g * kHeadDim;     // item = sequence x KV head
  const ChunkOut co{ch.item, ch.slot, ch.slot0, ch.nslots};
  float* s_ml = reinterpret_cast<float*>(smem);
  float* s_acc = s_ml + ml_lds_floats(NWV, HS);     // finish_lds_floats(NWV, g)
  if constexpr (LOOK) {
    if (ch.tier == kTierMerge) {
      merge::merge_part<NWV>(ma, ch);
      return;
    }
  }
  uint32_t state = merge::kAbsent;
  if (ch.tier == kTierTail) {   // appended tokens: 64-token tiles of bf16 rows, as many rows as exist so far
    const int rows = max(0, min(ch.rows, n_tail - ch.row0));
    state = process_tail_tiles<HS, false, NWV, LOOK>(arena + ch.k_data, arena + ch.v_data, rows, g, qp, s_ml, s_acc, ma, co);
    if constexpr (MULTI) return;
  } else if constexpr (!MULTI) {
#define RDKV_ONE(TIER_)                                                                                           \
  {                                                                                                               \
    Run<HS> run;                                                                                                  \
    run.init();                                                                                                   \
    process_tiles<TIER_, HS, NWV, ROOMY>(arena + ch.k_data, arena + ch.k_meta, arena + ch.v_data, arena + ch.v_meta,     \
                                  ch.rows, g, qp, run);                                                           \
    state = finish_chunk<HS, false, NWV, LOOK>(run, 16777216.0f, 0.f, g, s_ml, s_acc, ma, co);                           \
  }
    switch (ch.tier) {
      case 16:                  // (launches without 16-bit chunks get less LDS)
        if constexpr (ROOMY)
          state = process_rows_mfma<HS, true, NWV, LOOK>(arena + ch.k_data, arena + ch.v_data, ch.rows, g, qp, smem,
                                                         nullptr, nullptr, &ma, &co);
        break;
      case 8: RDKV_ONE(8) break;
      case 4: RDKV_ONE(4) break;
      default: RDKV_ONE(2) break;
    }
#undef RDKV_ONE
  }
  if constexpr (LOOK) merge::merge_left<NWV>(ma, co.item, co.slot0, co.nslots, state);
  if constexpr (!MULTI) return;
  // The workgroup's pieces: runs of rows of the item's quantized tiers on one softmax state.  A share of an item's
  // work goes through the tiers in the order 2, 4, 8 bits, so the chain is at most three pieces long and the three
  // tier bodies follow each other in a straight line (a loop around a switch made the compiler spill the state).
  Run<HS> run;
  run.init();
#define RDKV_PIECE(TIER_)                                                                                         \
  if (ch.tier == (TIER_)) {                                                                                       \
    const int next = ch.next;                                                                                     \
    process_tiles<TIER_, HS, NWV, ROOMY>(arena + ch.k_data, arena + ch.k_meta, arena + ch.v_data, arena + ch.v_meta,     \
                                  ch.rows, g, qp, run);                                                           \
    if (next >= 0) {                                                                                              \
      ch = chunks[next];                                                                                          \
    } else {                                                                                                      \
      ch.tier = 0;                                                                                                \
    }                                                                                                             \
  }
  RDKV_PIECE(2)
  RDKV_PIECE(4)
  RDKV_PIECE(8)
#undef RDKV_PIECE
  // ---- undo the subnormal unit, add the offsets, merge the wavefronts, hand the partial over -------------------
  finish_chunk<HS, false, NWV, LOOK>(run, 16777216.0f, 0.f, g, s_ml, s_acc, ma, co);
}

template <int HS, int NWV, bool MULTI, bool ROOMY, bool LOOK>
hipError_t launch_tiles(const Chunk* chunks, int first, int n_blocks, bool rows16, const uint8_t* arena, const uint16_t* q,
                        const MergeArgs& ma, const int32_t* tail_len, hipStream_t st) {
  size_t lds = (ml_lds_floats(NWV, HS) + finish_lds_floats(NWV, ma.g)) * sizeof(float);
  if constexpr (ROOMY)
    if (rows16) {
      constexpr size_t kRows = rows_lds_bytes<HS, NWV>();
      hipError_t e = RDKV_ALLOW_LDS((decode_tiles_kernel<HS, NWV, MULTI, ROOMY, LOOK>), kRows);
      if (e != hipSuccess) return e;
      lds = lds > kRows ? lds : kRows;
    }
  hipLaunchKernelGGL((decode_tiles_kernel<HS, NWV, MULTI, ROOMY, LOOK>), dim3(n_blocks), dim3(NWV * 64), lds, st, chunks, arena, q,
                     tail_len, first, ma.g, ma);
  return hipGetLastError();
}

}  // namespace

bool decode_tiles_take_rows(int n_chunks, bool multi) { return !multi && n_chunks <= 256; }

hipError_t launch_decode_tiles(const Chunk* chunks, int first, int n_chunks, int n_merge, bool rows16, bool multi,
                               const uint8_t* arena, const uint16_t* q, const MergeArgs& ma, const int32_t* tail_len,
                               hipStream_t st) {
  if (n_chunks == 0) return hipSuccess;
  const bool look = ma.parts > 0, roomy = decode_tiles_take_rows(n_chunks, multi);
  if ((look || rows16) && !roomy) return hipErrorInvalidValue;
  // up to 4 query heads per KV head: one head set, workgroups of eight wavefronts; 8 heads: two head sets, workgroups of
  // four
#define RDKV_TILES(HS_, NWV_)                                                                                             \
  if (look) return launch_tiles<HS_, NWV_, false, true, true>(chunks, first, n_chunks + n_merge, rows16, arena, q, ma, tail_len, st); \
  if (roomy) return launch_tiles<HS_, NWV_, false, true, false>(chunks, first, n_chunks, rows16, arena, q, ma, tail_len, st);         \
  if (multi) return launch_tiles<HS_, NWV_, true, false, false>(chunks, first, n_chunks, false, arena, q, ma, tail_len, st); \
  return launch_tiles<HS_, NWV_, false, false, false>(chunks, first, n_chunks, false, arena, q, ma, tail_len, st);
  if (ma.g > 4) {
    RDKV_TILES(2, 4)
  }
  RDKV_TILES(1, 8)
#undef RDKV_TILES
}

}  // namespace rdkv
