// 16 x 16 matrix-core steps on operands that come straight from memory, for contractions with few rows: both operands
// are contiguous along the contraction, and a lane's 16-byte load is its whole share of one step.
//
// One step multiplies 64 bytes of each of 16 A rows by 64 bytes of each of 16 B rows: lane l holds the bytes
// 16 * (l / 16) .. + 15 of row l % 16 of either operand.  bf16: eight values, one v_mfma_f32_16x16x32_bf16.  fp32: four
// values; instruction j takes value j of every lane, so the contraction indices of the four v_mfma_f32_16x16x4_f32 are
// permuted the same way in A and in B.  Lane l receives C[m][n] for n = l % 16 (B row), m = 4 * (l / 16) + r (A row).
#pragma once
#include "common.h"

namespace meft {

template <typename T>
struct Mma16;

template <>
struct Mma16<bf16_t> {
  static __device__ __forceinline__ f32x4 step(u32x4 a, u32x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  }
};

template <>
struct Mma16<float> {
  static __device__ __forceinline__ f32x4 step(u32x4 a, u32x4 b, f32x4 c) {
    const f32x4 fa = __builtin_bit_cast(f32x4, a), fb = __builtin_bit_cast(f32x4, b);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(fa.x, fb.x, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(fa.y, fb.y, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(fa.z, fb.z, c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x4f32(fa.w, fb.w, c, 0, 0, 0);
  }
};

// acc[i][j] += A rows of tile i (row starts pa[i]) times B rows of tile j (pb[j]) over the 64-byte steps s0 .. s1 - 1
// of rows of `row_bytes` bytes (a multiple of 16).  pa, pb: this lane's row.  U steps' loads are in flight together.
template <typename T, int NA, int NB, int U>
__device__ __forceinline__ void mma16_rows(const char* const (&pa)[NA], const char* const (&pb)[NB], int s0, int s1,
                                           int row_bytes, f32x4 (&acc)[NA][NB]) {
  const int q16 = ((threadIdx.x & 63) >> 4) * 16;
  for (int s = s0; s < s1; s += U) {
    u32x4 a[U][NA], b[U][NB];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      // beyond the row or the range: any valid address; both values are then replaced by zeros (one of them an infinity
      // would make the product of the other's zero NaN)
      const int off = (s + u) * 64 + q16;
      const int at = off < row_bytes ? off : 0;
#pragma unroll
      for (int i = 0; i < NA; ++i) a[u][i] = *reinterpret_cast<const u32x4*>(pa[i] + at);
#pragma unroll
      for (int j = 0; j < NB; ++j) b[u][j] = *reinterpret_cast<const u32x4*>(pb[j] + at);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in = s + u < s1 && (s + u) * 64 + q16 < row_bytes;
      const u32x4 zero = {0u, 0u, 0u, 0u};
      u32x4 bv[NB];
#pragma unroll
      for (int j = 0; j < NB; ++j) bv[j] = in ? b[u][j] : zero;
#pragma unroll
      for (int i = 0; i < NA; ++i) {
        const u32x4 av = in ? a[u][i] : zero;
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = Mma16<T>::step(av, bv[j], acc[i][j]);
      }
    }
  }
}

}  // namespace meft
