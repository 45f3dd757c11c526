// Exact division by a number that is the same for many dividends, by multiplication.  Plain C++ but for the function
// attributes, so that a host program can check it.
#pragma once
#include <stdint.h>

#ifdef __HIPCC__
#define MEFT_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define MEFT_HOST_DEVICE inline
#endif

namespace meft {

// ceil(2^32 / m) for m > 1 (0 for m == 1, where tile_div does not use it).  No branch: it would differ per lane.
MEFT_HOST_DEVICE uint32_t tile_div_inverse(uint32_t m) { return 0xFFFFFFFFu / m + 1u; }

// w / m for 0 <= w < 2^31 and 1 <= m < 2^31.  inv = (2^32 + e) / m with 0 <= e < m, so w * inv / 2^32 is too large by
// w * e / (m * 2^32) < 1/2: its floor is the quotient or, from w * m around 2^32 on, one more.
MEFT_HOST_DEVICE int tile_div(int w, int m, uint32_t inv) {
  if (m == 1) return w;
  const int q = (int)(((uint64_t)(uint32_t)w * inv) >> 32);
  return (uint32_t)q * (uint32_t)m > (uint32_t)w ? q - 1 : q;
}

}  // namespace meft
