// Pieces that the bf16-fragment step kernels (banded_wide.hip, banded_direct.hip) share: bit bytes as matrix-core
// operands and the feature order of their staged slices.
#pragma once

#include "device_common.h"

namespace ggnn {
namespace dev {

// Row of feature f of a 32-feature group, as 16 * tile + row: tile 2j + i of
// group j holds features 32j + 8r + 4i + {0..3} in rows 4r + {0..3}, so that a
// lane's sums of two tiles are eight consecutive features (a fragment of the
// transform, weight rows read 16 bytes at a time, one 16-byte store of dM).
__device__ __forceinline__ int feature_slot(int f) {
  const int w = f % 32;
  return 32 * (f / 32) + 16 * ((w % 8) / 4) + 4 * (w / 8) + w % 4;
}

// 8 bits -> 8 bf16 elements equal to 0 or 1 (bit i -> element i).
__device__ __forceinline__ bf16x8 bits_frag(uint32_t byte) {
  const uint32_t x = byte * 0x8001u;
  u32x4 w;
#pragma unroll
  for (int k = 0; k < 4; ++k) w[k] = (x & (0x10001u << (2 * k))) * (0x3F80u >> (2 * k));
  return __builtin_bit_cast(bf16x8, w);
}

// Whether any lane of the wave holds a nonzero x (the same answer in every
// lane, so a branch on it is taken by the whole wave).
__device__ __forceinline__ bool wave_any(uint32_t x) { return __builtin_amdgcn_ballot_w64(x != 0u) != 0; }

}  // namespace dev
}  // namespace ggnn
