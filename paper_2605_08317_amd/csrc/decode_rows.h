// Split-K flash-decode over row-major bf16 rows (Sec. 3.3, Eq. 7) on the gfx950 matrix cores: the uncompressed path
// (the full-cache baseline of Sec. 4.2) and the 16-bit tier of a token-wise cache.
//
// Caller-owned rows are row-major [token][128 channels], so a coalesced load hands a lane 8 channels of one token,
// while the 4x4x4 products want a lane to be a token on the K side (4 consecutive channels per step) and a channel
// on the V side (4 consecutive tokens per step).  Each wavefront therefore passes its 64-token tiles through a
// region of LDS of its own: 16 coalesced 16-byte loads per lane and side, stored row by row with a row stride of 272
// bytes (so that the 16 lanes that read their own rows at the same column hit different banks), then
//   q K^T   lane = token reads its row back: A = the raw bf16 query (exact products), broadcast from the lanes that hold
//           a step's channels, B = 4 channels of the token, D: lane = token, turned to lane (block b, head j);
//   P V     lane = channel pair (2 lane, 2 lane + 1) reads one 32-bit word per token: two byte permutes make the
//           B operands of 4 consecutive tokens for the even and the odd channel; A = the probabilities of those 4
//           tokens as two truncated bf16 terms, broadcast from the block that holds them (cbsz = 4).
// The V loads of a tile are in flight while its logits are computed, the next tile's K loads during P V.  With 8
// query heads per KV head the plain-ALU kernel this replaces spent 2 x 8 multiply-adds per loaded element; here the
// per-element work is one LDS write, one LDS read and a fraction of a byte permute, whatever the number of heads.
#pragma once
#include <utility>

#include "decode_tile_common.h"

namespace rdkv {
namespace tile {

constexpr int kRowStride = 272;                       // bytes per token row in LDS (256 + 16 of padding)
constexpr int kStageBytes = kTile * kRowStride;       // one wavefront's staging region
template <int HS, int NWV>
constexpr int rows_lds_bytes() {
  // the wavefronts' staging regions, their maxima and sums;
  // the end-of-chunk areas (per-wavefront accumulators [waves][g][128] floats, then the merge) reuse the staging
  return NWV * kStageBytes + ml_lds_floats(NWV, HS) * 4;
}

__device__ __forceinline__ uint4 load_row_chunk(const uint8_t* __restrict__ base, int row, int c16) {
  return *reinterpret_cast<const uint4*>(base + static_cast<int64_t>(row) * (kHeadDim * 2) + c16 * 16);
}

// One step of P V: tokens 4 A .. 4 A + 3 (A is an instruction field, hence a template argument).
template <int A, int HS>
__device__ __forceinline__ void pv_step(const uint8_t* s_stage, int lane, const short4v (&phi)[HS],
                                        const short4v (&plo)[HS], Run<HS>& run) {
  uint32_t w[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) w[k] = *reinterpret_cast<const uint32_t*>(s_stage + (4 * A + k) * kRowStride + 4 * lane);
  // low halves of two tokens' words = the even channel, high halves = the odd channel
  const short4v be = bf4(__builtin_amdgcn_perm(w[1], w[0], 0x05040100u), __builtin_amdgcn_perm(w[3], w[2], 0x05040100u));
  const short4v bo = bf4(__builtin_amdgcn_perm(w[1], w[0], 0x07060302u), __builtin_amdgcn_perm(w[3], w[2], 0x07060302u));
#pragma unroll
  for (int hs = 0; hs < HS; ++hs) {
    run.acc[hs][0] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(phi[hs], be, run.acc[hs][0], 4, A, 0);
    run.acc[hs][0] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(plo[hs], be, run.acc[hs][0], 4, A, 0);
    run.acc[hs][1] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(phi[hs], bo, run.acc[hs][1], 4, A, 0);
    run.acc[hs][1] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(plo[hs], bo, run.acc[hs][1], 4, A, 0);
  }
}
template <int HS, int... A>
__device__ __forceinline__ void pv_steps(const uint8_t* s_stage, int lane, const short4v (&phi)[HS],
                                         const short4v (&plo)[HS], Run<HS>& run, std::integer_sequence<int, A...>) {
  (pv_step<A, HS>(s_stage, lane, phi, plo, run), ...);
}

// TIERED: the chunk's partial goes to the split workspace for the launch's merging workgroups (LOOK) or is announced
// (store_partial); otherwise it is only stored, for a launch that follows or (THROUGH: to memory) merge_tagged.
template <int HS, bool TIERED, int NWV, bool LOOK = false, bool THROUGH = false>
__device__ __forceinline__ uint32_t process_rows_mfma(const uint8_t* __restrict__ kd, const uint8_t* __restrict__ vd,
                                                  int rows, int g, const uint16_t* __restrict__ q, uint8_t* smem,
                                                  float* __restrict__ part_acc, float* __restrict__ part_ml,
                                                  const MergeArgs* ma, const ChunkOut* co) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int blk = lane >> 2, j = lane & 3;
  uint8_t* s_stage = smem + wave * kStageBytes;
  float* s_ml = reinterpret_cast<float*>(smem + NWV * kStageBytes);
  float* s_acc = reinterpret_cast<float*>(smem);   // after the tile loop: [waves][g][128], then the merge
  const int ntiles = (rows + kTile - 1) / kTile;
  const int last = rows - 1;
  const int lr = lane >> 4, lc = lane & 15;            // a load covers 4 rows x 16 chunks of 16 bytes

  uint4 st[16];
  auto load_tile = [&](const uint8_t* __restrict__ base, int t) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 16; ++i) st[i] = load_row_chunk(base, min(t * kTile + 4 * i + lr, last), lc);
  };
  auto store_tile = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 16; ++i) *reinterpret_cast<uint4*>(s_stage + (4 * i + lr) * kRowStride + 16 * lc) = st[i];
  };
  uint4 qa[HS];      // the query on the A side, raw bf16 (exact products); loads return in order, so it goes first
#pragma unroll
  for (int hs = 0; hs < HS; ++hs) qa[hs] = load_query(q, 4 * hs + j, g, blk);
  if (wave < ntiles) load_tile(kd, wave);

  Run<HS> run;
  run.init();
  const floatx4 zero4 = {0.f, 0.f, 0.f, 0.f};
  for (int tile = wave; tile < ntiles; tile += NWV) {
    const int next = tile + NWV;
    store_tile();                       // K rows of this tile (the loads were issued a tile ago)
    load_tile(vd, tile);                // V rows: in flight during the logits
    wave_lds_sync();
    floatx4 a16[HS];
#pragma unroll
    for (int hs = 0; hs < HS; ++hs) a16[hs] = zero4;
    // 16 bytes of the lane's own token row = 8 channels = block I's two steps
#define RDKV_ROWS_K(I_)                                                                                              \
  {                                                                                                                 \
    const uint4 kr = *reinterpret_cast<const uint4*>(s_stage + lane * kRowStride + 16 * (I_));                      \
    _Pragma("unroll") for (int hs = 0; hs < HS; ++hs) {                                                             \
      a16[hs] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(bf4(qa[hs].x, qa[hs].y), bf4(kr.x, kr.y), a16[hs], 4, I_, 0); \
      a16[hs] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(bf4(qa[hs].z, qa[hs].w), bf4(kr.z, kr.w), a16[hs], 4, I_, 0); \
    }                                                                                                               \
  }
    RDKV_ROWS_K(0) RDKV_ROWS_K(1) RDKV_ROWS_K(2) RDKV_ROWS_K(3) RDKV_ROWS_K(4) RDKV_ROWS_K(5) RDKV_ROWS_K(6)
    RDKV_ROWS_K(7) RDKV_ROWS_K(8) RDKV_ROWS_K(9) RDKV_ROWS_K(10) RDKV_ROWS_K(11) RDKV_ROWS_K(12) RDKV_ROWS_K(13)
    RDKV_ROWS_K(14) RDKV_ROWS_K(15)
#undef RDKV_ROWS_K
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

    wave_lds_sync();                    // every lane is done with the K rows
    store_tile();                       // V rows
    if (next < ntiles) load_tile(kd, next);   // the next tile's K rows: in flight during P V
    wave_lds_sync();
    // P V: step a = tokens 4a..4a+3; this lane's word of a token row = channels 2 lane, 2 lane + 1
    pv_steps<HS>(s_stage, lane, phi, plo, run, std::make_integer_sequence<int, 16>{});
    wave_lds_sync();                    // before the next tile's K rows overwrite the region
  }

  // ---- end of the chunk: merge the workgroup's wavefronts, store the partial ---------------------------------------
#pragma unroll
  for (int hs = 0; hs < HS; ++hs) run.l[hs] = head_sum(run.l[hs]);
  uint32_t state = merge::kAbsent;
  if constexpr (TIERED) state = ends_soon<LOOK, NWV>(g, *ma, *co);
  __syncthreads();                      // the staging regions become the accumulator area
#pragma unroll
  for (int hs = 0; hs < HS; ++hs) {
    if (lane < 16)        // (block, j) -> group block of head j; log2 domain from here on
      *reinterpret_cast<float4*>(s_ml + ml_at<HS>(wave, 4 * hs + (lane & 3), lane >> 2)) =
          make_float4(run.m[hs] * kXScale - kPExp, run.l[hs], 0.f, 0.f);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int head = 4 * hs + i;
      if (head < g)
        *reinterpret_cast<float2*>(s_acc + (wave * g + head) * kHeadDim + 2 * lane) =
            make_float2(run.acc[hs][0][i], run.acc[hs][1][i]);
    }
  }
  if constexpr (TIERED) {
    store_partial<HS, NWV, LOOK>(1.0f, g, s_ml, s_acc, *ma, *co);
  } else {
    __syncthreads();
    for (int idx = tid; idx < g * kHeadDim; idx += NWV * 64) {
      const int head = idx >> 7;
      float m[NWV], mm = kNegBig, v = 0.f, ll = 0.f;
#pragma unroll
      for (int w = 0; w < NWV; ++w) {
        m[w] = s_ml[ml_at<HS>(w, head, 0)];
        mm = fmaxf(mm, m[w]);
      }
#pragma unroll
      for (int w = 0; w < NWV; ++w) {
        const float f = fast_exp2(m[w] - mm);
        v = __builtin_fmaf(s_acc[w * g * kHeadDim + idx], f, v);
        ll = __builtin_fmaf(s_ml[ml_at<HS>(w, head, 0) + 1], f, ll);
      }
      if constexpr (THROUGH) merge::store_agent(part_acc + idx, v); else part_acc[idx] = v;
      if ((idx & 127) == 0) {
        if constexpr (THROUGH) {
          merge::store_agent(part_ml + head * 2, mm);
          merge::store_agent(part_ml + head * 2 + 1, ll);
        } else {
          part_ml[head * 2] = mm;
          part_ml[head * 2 + 1] = ll;
        }
      }
    }
  }
  return state;
}

}  // namespace tile
}  // namespace rdkv
