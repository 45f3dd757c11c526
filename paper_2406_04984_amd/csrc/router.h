// Router scores (Eq. 5) as a skinny contraction without LDS tiles, and the top-e selection over partial scores
// (Algorithm 1: tau <- TopK(p, number of experts)).
#pragma once
#include "mma16.h"

namespace meft {

constexpr int kRouteWaves = 8;

// p[part][t][b] = partial score of token t and block b over slice `part` of the hidden dimension.  A workgroup takes 16
// tokens * TT, 16 blocks * NA and one of the n_part slices, which its eight waves share out again; each multiplies with
// 16 x 16 matrix-core steps straight from memory, and the waves are added through LDS in order.
// Grid: (ceil(B / (16 * NA)) * ceil(T / (16 * TT)), 1, n_part), the blocks fastest (a batch has more token tiles than a
// launch may have workgroups along y).
//
// Used as long as the problem is small (route_on_tiles has the lines): what bounds it there is the latency of a compute
// unit's loads (one compute unit has about a hundred 128-byte lines in flight, so one alone takes 12 us to read the router
// of a 4096 x 64 layer), and the LDS-tiled contractions (ProbRouter, gemm_nt.h) fill too few of them and pay for their
// ring's start.  For large problems the tiled ones move a fraction of the bytes per flop.
template <typename T, int NA, int TT>
__global__ __launch_bounds__(64 * kRouteWaves) void route_part_kernel(const T* __restrict__ h, const T* __restrict__ Wg,
                                                                      int n_tok, int d, int B, float* __restrict__ p) {
  __shared__ __attribute__((aligned(16))) float s_part[kRouteWaves][NA][TT][64][4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int b_tiles = (B + 16 * NA - 1) / (16 * NA), t_tile = blockIdx.x / b_tiles;
  const int b0 = (blockIdx.x - t_tile * b_tiles) * 16 * NA, t0 = t_tile * 16 * TT;
  const int row_bytes = d * (int)sizeof(T);
  const char *pa[NA], *pb[TT];
#pragma unroll
  for (int i = 0; i < NA; ++i) pa[i] = reinterpret_cast<const char*>(Wg + (size_t)min(b0 + i * 16 + (lane & 15), B - 1) * d);
#pragma unroll
  for (int j = 0; j < TT; ++j) pb[j] = reinterpret_cast<const char*>(h + (size_t)min(t0 + j * 16 + (lane & 15), n_tok - 1) * d);
  f32x4 acc[NA][TT];
#pragma unroll
  for (int i = 0; i < NA; ++i)
#pragma unroll
    for (int j = 0; j < TT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int steps = (row_bytes + 63) / 64, n_slice = (int)gridDim.z * kRouteWaves;
  const int per = (steps + n_slice - 1) / n_slice, slice = blockIdx.z * kRouteWaves + wave;
  mma16_rows<T, NA, TT, 4>(pa, pb, min(steps, slice * per), min(steps, (slice + 1) * per), row_bytes, acc);
#pragma unroll
  for (int i = 0; i < NA; ++i)
#pragma unroll
    for (int j = 0; j < TT; ++j) *reinterpret_cast<f32x4*>(&s_part[wave][i][j][lane][0]) = acc[i][j];
  __syncthreads();
  for (int x = tid; x < NA * TT * 64; x += 64 * kRouteWaves) {
    const int l = x & 63, j = (x >> 6) % TT, i = (x >> 6) / TT;
    f32x4 v = *reinterpret_cast<const f32x4*>(&s_part[0][i][j][l][0]);
#pragma unroll
    for (int w = 1; w < kRouteWaves; ++w) v += *reinterpret_cast<const f32x4*>(&s_part[w][i][j][l][0]);
    const int t = t0 + j * 16 + (l & 15), b = b0 + i * 16 + (l >> 4) * 4;
    if (t >= n_tok) continue;
    float* o = p + ((size_t)blockIdx.z * n_tok + t) * B + b;
    if ((B & 3) == 0) {
      if (b < B) *reinterpret_cast<f32x4*>(o) = v;
    } else {
#pragma unroll
      for (int z = 0; z < 4; ++z)
        if (b + z < B) o[z] = v[z];
    }
  }
}

// largest value of the wave, in every lane
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
#define MEFT_DPP_MAX(ctrl, rows) \
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, ctrl, rows, 0xF, false))
  MEFT_DPP_MAX(0xB1, 0xF);    // quad_perm [1,0,3,2]
  MEFT_DPP_MAX(0x4E, 0xF);    // quad_perm [2,3,0,1]
  MEFT_DPP_MAX(0x141, 0xF);   // row_half_mirror
  MEFT_DPP_MAX(0x140, 0xF);   // row_mirror: every lane holds its row's maximum
  MEFT_DPP_MAX(0x142, 0xA);   // row_bcast:15 into rows 1 and 3
  MEFT_DPP_MAX(0x143, 0xC);   // row_bcast:31 into rows 2 and 3: row 3 holds the wave's maximum
#undef MEFT_DPP_MAX
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Top-e blocks of up to 64 * Z blocks, one wave per token, four tokens per workgroup.  Lane l keeps the keys of the
// blocks l, l + 64, ... in registers; e rounds of a wave-wide maximum through DPP moves, its lowest block by ballots,
// and the winner is retired by zeroing its key (a live key is never 0 for finite scores).  Output order: score
// descending, block id ascending.  Against keys in LDS and 64-bit shuffles: 8.7 -> 5 us (8192 tokens, 64 blocks).
template <int Z>
__global__ __launch_bounds__(256) void route_pick_kernel(const float* __restrict__ p, int n_part, size_t part_stride,
                                                         const float* __restrict__ bias, int n_tok, int B, int e,
                                                         int32_t* __restrict__ block_idx, float* __restrict__ block_score) {
  const int lane = threadIdx.x & 63, t = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= n_tok) return;
  const float* row = p + (size_t)t * B;
  uint32_t key[Z];
#pragma unroll
  for (int z = 0; z < Z; ++z) {
    const int b = z * 64 + lane;
    key[z] = 0u;
    if (b < B) {
      float v = row[b];
      for (int s = 1; s < n_part; ++s) v += row[s * part_stride + b];   // partial scores of a split contraction
      if (bias) v += bias[b];
      key[z] = order_key(v);
    }
  }
  for (int q = 0; q < e; ++q) {
    uint32_t best = key[0];
#pragma unroll
    for (int z = 1; z < Z; ++z) best = max(best, key[z]);
    best = wave_max_u32(best);
    int sel = 0;   // lowest block with that key
#pragma unroll
    for (int z = Z - 1; z >= 0; --z) {
      const unsigned long long m = __ballot(key[z] == best);
      if (m) sel = z * 64 + __ffsll(m) - 1;
    }
    sel = min(sel, B - 1);
#pragma unroll
    for (int z = 0; z < Z; ++z)
      if (sel == z * 64 + lane) key[z] = 0u;
    if (lane == 0) {
      block_idx[(size_t)t * e + q] = sel;
      if (block_score) block_score[(size_t)t * e + q] = key_to_float(best);
    }
  }
}

}  // namespace meft
