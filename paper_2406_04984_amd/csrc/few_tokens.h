// The forward for few tokens (decoding batches): up to kFewEntries (token, block) entries.  With so few entries the
// time is launches, chains of small index kernels, and the reads of the blocks' keys, so the forward is two launches
// and no index structure:
//   few_score    one workgroup per (block in use, 16 * NA of its neurons): finds the tokens of the block by looking
//                through all entries, and scores them (Eq. 6) with 16 x 16 matrix-core steps straight from memory, the
//                hidden dimension shared out over its eight waves;
//   few_out      one workgroup per (token, columns of its output row): the token's top-k selection -- repeated by each
//                of the token's workgroups, it costs less than a launch -- then the selected value rows are summed pair
//                by pair in fp32 (Eq. 1-4).
// Both element types.  Measured at the LLaMA-7B-shaped layer (64 blocks of 1024, top_e 4, top_k 256), route and forward
// together, against the eleven launches of the block-dense path: 1 token 101 -> 23 us with its 35 MB of weights in the caches,
// 148 -> 68 us on a layer not used before; 24 tokens 196 -> 107 us (the keys of the ~50 blocks in use are 0.42 GB, 91 us at the
// 4.6 TB/s of a copy).  At the limit, forward alone, 128 tokens of 4 blocks: 248 -> 162 us (129 tokens, on the other path, take
// 185); 128 tokens of a 64 x 256 x 1024 layer 79 -> 19 (129: 47); 64 tokens of 8 of 64 x 96 x 4096 113 -> 28 (65: 63).
#pragma once
#include "mma16.h"
#include "select.h"

namespace meft {

constexpr int kFewEntries = 512;      // entries (tokens x top_e) of the batch: one thread of few_score each
constexpr int kFewWaves = 8;
constexpr int kFewMaxE = 64;

// The row of the score matrix that entry (t, q) of block b owns: rows of a token are in ascending block order.
__device__ __forceinline__ int few_rank(const int32_t* __restrict__ tok_blocks, int e, int n_blocks, int b, int q) {
  int r = 0;
  for (int z = 0; z < e; ++z) {
    const int bz = clampi(tok_blocks[z], 0, n_blocks - 1);
    r += (bz < b || (bz == b && z < q)) ? 1 : 0;
  }
  return r;
}

// Grid: (ceil(bs / (16 * NA)), by_block ? n_blocks : n_ent).  Row y is a block, or an entry whose workgroups go on only
// if it is the first entry of its block (fewer entries than blocks).
template <typename T, int NA>
__global__ __launch_bounds__(64 * kFewWaves) void few_score_kernel(const T* __restrict__ h, const T* __restrict__ K,
                                                                   const int32_t* __restrict__ block_idx, int n_ent, int e,
                                                                   int n_blocks, int bs, int d, int by_block,
                                                                   float* __restrict__ sc) {
  __shared__ int s_list[kFewEntries];   // entries of the block, ascending; then the score rows they own
  __shared__ int s_tok[kFewEntries];
  __shared__ int s_cnt[kFewWaves];
  __shared__ __attribute__((aligned(16))) float s_part[kFewWaves][NA][64][4];
  static_assert(kFewEntries == 64 * kFewWaves, "one thread per entry");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int b = by_block ? (int)blockIdx.y : clampi(block_idx[blockIdx.y], 0, n_blocks - 1);
  const bool hit = tid < n_ent && clampi(block_idx[min(tid, n_ent - 1)], 0, n_blocks - 1) == b;
  const unsigned long long m = __ballot(hit);
  if (lane == 0) s_cnt[wave] = __popcll(m);
  __syncthreads();
  int n = 0, at = 0;
#pragma unroll
  for (int w = 0; w < kFewWaves; ++w) { const int c = s_cnt[w]; at += w < wave ? c : 0; n += c; }
  if (hit) s_list[at + __popcll(m & ((1ull << lane) - 1ull))] = tid;
  __syncthreads();
  if (n == 0 || (!by_block && s_list[0] != (int)blockIdx.y)) return;
  int row = 0, tok = 0;
  if (tid < n) {
    const int ent = s_list[tid];
    tok = ent / e;
    row = tok * e + few_rank(block_idx + (size_t)tok * e, e, n_blocks, b, ent - tok * e);
  }
  __syncthreads();
  if (tid < n) { s_list[tid] = row; s_tok[tid] = tok; }
  __syncthreads();

  const int r0 = blockIdx.x * 16 * NA;   // first neuron, inside the block
  const int row_bytes = d * (int)sizeof(T);
  const int steps = (row_bytes + 63) / 64, per = (steps + kFewWaves - 1) / kFewWaves;
  const int s0 = wave * per, s1 = min(steps, s0 + per);
  const char* pa[NA];
#pragma unroll
  for (int i = 0; i < NA; ++i)
    pa[i] = reinterpret_cast<const char*>(K + ((size_t)b * bs + min(r0 + i * 16 + (lane & 15), bs - 1)) * d);
  auto tile = [&](auto nt_tag, int base) {   // tokens base .. base + 16 * NT - 1 of the list
    constexpr int NT = decltype(nt_tag)::value;
    const char* pb[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j)
      pb[j] = reinterpret_cast<const char*>(h + (size_t)s_tok[min(base + j * 16 + (lane & 15), n - 1)] * d);
    f32x4 acc[NA][NT];
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // two steps of loads in flight per wave: more keep fewer waves on a compute unit, which costs more (24 tokens: 107
    // us with two steps, 115 with four, 132 with eight)
    mma16_rows<T, NA, NT, 2>(pa, pb, s0, s1, row_bytes, acc);
#pragma unroll
    for (int j = 0; j < NT; ++j) {
#pragma unroll
      for (int i = 0; i < NA; ++i) *reinterpret_cast<f32x4*>(&s_part[wave][i][lane][0]) = acc[i][j];
      __syncthreads();
      if (tid < 64 * NA) {   // item: tile i, lane l of the accumulator layout; the waves are added in order
        const int i = tid >> 6, l = tid & 63;
        f32x4 v = *reinterpret_cast<const f32x4*>(&s_part[0][i][l][0]);
#pragma unroll
        for (int w = 1; w < kFewWaves; ++w) v += *reinterpret_cast<const f32x4*>(&s_part[w][i][l][0]);
        const int x = base + j * 16 + (l & 15), r = r0 + i * 16 + (l >> 4) * 4;
        if (x < n) {
          float* o = sc + (size_t)s_list[x] * bs + r;
          if ((bs & 3) == 0) {
            if (r < bs) *reinterpret_cast<f32x4*>(o) = v;
          } else {
#pragma unroll
            for (int z = 0; z < 4; ++z)
              if (r + z < bs) o[z] = v[z];
          }
        }
      }
      __syncthreads();
    }
  };
  for (int base = 0; base < n; base += 32) {
    if (n - base > 16) tile(std::integral_constant<int, 2>{}, base);
    else tile(std::integral_constant<int, 1>{}, base);
  }
}

// Grid: (ceil(d / (8 * CL)), T), or (1, T) with out == nullptr (selection only).  CL lanes cover the workgroup's
// columns, eight each; the 256 / CL groups of CL threads share out the pairs and are added in group order.
template <typename T, int KPT, bool kFull, int CL>
__global__ __launch_bounds__(256) void few_out_kernel(const float* __restrict__ sc, const int32_t* __restrict__ block_idx,
                                                      const T* __restrict__ V, int C, int bs, int e, int k, int n_blocks,
                                                      int d, int32_t* __restrict__ idx, float* __restrict__ act,
                                                      T* __restrict__ out) {
  constexpr int G = 256 / CL, NC = CL * 8;
  __shared__ TopkLds s;
  __shared__ int s_blk[kFewMaxE];
  __shared__ float s_red[G][NC];
  const int t = blockIdx.y, tid = threadIdx.x;
  if (tid < e) {
    const int32_t* tb = block_idx + (size_t)t * e;
    const int b = clampi(tb[tid], 0, n_blocks - 1);
    s_blk[few_rank(tb, e, n_blocks, b, tid)] = b;
  }
  const int p0 = tid * KPT;
  {
    uint32_t key[KPT];
    topk_load_keys<KPT>(sc + (size_t)t * C, C, p0, key);
    uint32_t thr, sel = 0u, sel_hi = 0u;
    int need, gt_before, eq_before;
    topk_threshold<KPT, kFull>(key, C, p0, k, s, thr, need);
    topk_counts_before<KPT, kFull>(key, C, p0, thr, s, gt_before, eq_before);
    topk_stage<KPT, kFull>(key, C, p0, thr, need, gt_before, eq_before, 0, s, sel, sel_hi);   // k <= kTopkEmitLds
  }
  __syncthreads();
  for (int j = tid; j < k; j += 256) {
    const int i = s.idx[j], q = i / bs;
    const int nid = s_blk[q] * bs + (i - q * bs);
    const float v = key_to_float(__float_as_uint(s.act[j])), a = v > 0.f ? v : 0.f;
    s.idx[j] = nid;
    s.act[j] = a;
    if (blockIdx.x == 0) {
      idx[(size_t)t * k + j] = nid;
      act[(size_t)t * k + j] = a;
    }
  }
  if (out == nullptr) return;
  __syncthreads();
  const int g = tid / CL, cl = tid % CL;
  const int col = blockIdx.x * NC + cl * 8;
  float acc[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) acc[c] = 0.f;
  if (col < d) {
    constexpr int U = 8;
    int j = g;
    for (; j + G * (U - 1) < k; j += G * U) {
      float x[U][8];
#pragma unroll
      for (int u = 0; u < U; ++u) Vec8<T>::load(V + (size_t)s.idx[j + G * u] * d + col, x[u]);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float a = s.act[j + G * u];
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[c] = fmaf(a, x[u][c], acc[c]);
      }
    }
    for (; j < k; j += G) {
      float x[8];
      Vec8<T>::load(V + (size_t)s.idx[j] * d + col, x);
      const float a = s.act[j];
#pragma unroll
      for (int c = 0; c < 8; ++c) acc[c] = fmaf(a, x[c], acc[c]);
    }
  }
  Vec8<float>::store(&s_red[g][cl * 8], acc);
  __syncthreads();
  if (tid < CL && col < d) {
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[c] = s_red[0][tid * 8 + c];
    for (int z = 1; z < G; ++z)
#pragma unroll
      for (int c = 0; c < 8; ++c) acc[c] += s_red[z][tid * 8 + c];
    Vec8<T>::store(out + (size_t)t * d + col, acc);
  }
}

}  // namespace meft
