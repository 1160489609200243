// Geometry of the matrix-core attention kernel (attention_mfma.hip) that the
// split rule (api.hip) needs too: LDS layout, staging bounds, resident waves.
#pragma once

#include "attn_common.h"

namespace mf {

// Bytes of the selector table: entry n (a bitmap nibble) holds the byte
// selectors of channel pairs (0, 1) and (2, 3), 8 bytes.
constexpr uint32_t kLutBytes = 128;
// Value entries: a u32 per (token, column of 4 T channels), 16 per token, rows
// padded so that the rows of tokens 4 apart start 16 banks apart.
constexpr uint32_t kEntRow = 80;
constexpr uint32_t kColRow = 4u * kWave;  // bytes per key row: one dword per tile of the block

template <int T>
struct MfmaGeom {
  static constexpr int NB = kWave / T;        // tokens per block
  static constexpr int NG = NB / 16;          // 16-token groups per block
  static constexpr int NC = 2 * T;            // score MFMAs (8 channels per quad) per group
  static constexpr int NO = 4 * T;            // channels per column, O accumulators
};

// Byte offsets in the workgroup's LDS. The kernel has no static LDS, so they are
// LDS addresses (the selector table is at 0).
struct MfmaLds {
  uint32_t ent, kv, total;
};

// [table][entries][keys of the block, then its values]: key columns need 8 rows
// per 16-byte piece of a tile and two rows that the last nibble's second dword
// may touch; values a dword each plus the same two and what a whole piece of
// 512 writes past them.
template <int T>
__host__ __device__ inline MfmaLds mfma_lds_layout(int kpieces, int vchunks) {
  MfmaLds L;
  L.ent = kLutBytes;
  L.kv = L.ent + MfmaGeom<T>::NB * kEntRow;
  const uint32_t a = (8u * kpieces + 3u) * kColRow;
  const uint32_t b = (uint32_t)vchunks * kChunk * 4u + 16u;
  L.total = L.kv + (a > b ? a : b);
  return L;
}

// Most 16-byte pieces of a key tile, and 512-value chunks of a block's value run.
inline void mfma_staging(int T, const SparseSide& K, const SparseSide& V, int* kp, int* vc) {
  const int tile = K.group_keep >= 0 || K.n_keep > kTile ? kTile : K.n_keep;
  *kp = tile > 8 ? (tile + 7) / 8 : 1;
  const int run = side_token_bound(kTile * T, V, kWave / T) * (kWave / T);
  *vc = run > (int)kChunk ? (run + (int)kChunk - 1) / (int)kChunk : 1;
}

// Waves per SIMD that an instance's register budget is set for: three (168
// VGPRs) with the smaller key staging, else two. With three the larger instances
// spill: 1491 us against 757 on 512 streams of 32K tokens at K 50% / V 70%.
constexpr int mfma_waves(int T, int KP) { return T <= 2 && KP <= 5 ? 3 : 2; }

// Waves of the kernel that a CU holds at once, by LDS and registers.
inline int mfma_resident_waves(int T, const SparseSide& K, const SparseSide& V) {
  int kp, vc;
  mfma_staging(T, K, V, &kp, &vc);
  const uint32_t lds = T == 1 ? mfma_lds_layout<1>(kp, vc).total
                     : T == 2 ? mfma_lds_layout<2>(kp, vc).total
                              : mfma_lds_layout<4>(kp, vc).total;
  const int by_lds = (int)((160u << 10) / lds), by_regs = 4 * mfma_waves(T, kp <= 5 && vc <= 3 ? 5 : 8);
  return by_lds < by_regs ? by_lds : by_regs;
}

}  // namespace mf
