// Score GEMMs: C[m, n] = sum_c A[row(m), c] * Bm[n, c]  ("NT": both operands are contiguous
// along the contraction).  Used for the router scores (Eq. 5: one problem, A = h, Bm = Wg) and
// for the in-block key scores (Eq. 6: one problem per block, rows = the tokens routed to the
// block, Bm = that block's keys).  fp32 accumulation.
#pragma once
#include "common.h"

namespace meft {

struct GemmNTArgs {
  const void* A;         // rows of length Kdim, leading dimension lda
  const void* Bm;        // [n_groups*Ng, ldb]; group g owns rows [g*Ng, (g+1)*Ng)
  float* C;              // output rows, leading dimension ldc
  const int* perm;       // entries grouped by problem ([group_off[n_groups]]), or nullptr
  const int* group_off;  // [n_groups+1] first slot of each group in perm, or nullptr
  const int* tile_off;   // [n_groups+1] prefix sum of ceil(rows_g / BM), or nullptr
  int n_groups;          // 1 when perm == nullptr
  int M;                 // rows when perm == nullptr
  int Ng;                // columns per group
  int Kdim;
  int lda, ldb, ldc;
  int e;                 // with perm: A row = entry / e, C row = entry
};

// Finds the group and the first row of m-tile `mt`; returns false if the tile does not exist.
template <int BM>
__device__ __forceinline__ bool locate_tile(const GemmNTArgs& a, int mt, int& g, int& m0, int& Mg,
                                            int& slot0) {
  if (a.perm == nullptr) {
    g = 0; m0 = mt * BM; Mg = a.M; slot0 = 0;
    return m0 < Mg;
  }
  if (mt >= a.tile_off[a.n_groups]) return false;
  int lo = 0, hi = a.n_groups;  // tile_off[lo] <= mt < tile_off[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (a.tile_off[mid] <= mt) lo = mid; else hi = mid;
  }
  g = lo;
  m0 = (mt - a.tile_off[g]) * BM;
  slot0 = a.group_off[g];
  Mg = a.group_off[g + 1] - slot0;
  return true;
}

// ---------------------------------------------------------------------------------------------
// bf16 inputs, MFMA 32x32x16, 128x128 tile, 4 waves (2x2), each wave 64x64 = 2x2 MFMA tiles.
// LDS rows are padded by 8 elements (16 B) so that the 32 rows an operand read touches start in
// different banks.
// ---------------------------------------------------------------------------------------------
constexpr int kGemmBM = 128, kGemmBN = 128, kGemmBK = 64, kGemmPad = 8;

__global__ __launch_bounds__(256) void gemm_nt_bf16_kernel(GemmNTArgs a) {
  constexpr int BM = kGemmBM, BN = kGemmBN, BK = kGemmBK, LD = kGemmBK + kGemmPad;
  __shared__ __attribute__((aligned(16))) uint16_t sA[BM * LD];
  __shared__ __attribute__((aligned(16))) uint16_t sB[BN * LD];
  __shared__ int sRowA[BM];
  __shared__ int sRowC[BM];

  int g, m0, Mg, slot0;
  if (!locate_tile<BM>(a, blockIdx.x, g, m0, Mg, slot0)) return;
  const int n0 = blockIdx.y * BN;
  const int tid = threadIdx.x;

  if (tid < BM) {
    const int m = m0 + tid;
    int ra = -1, rc = -1;
    if (m < Mg) {
      if (a.perm) { rc = a.perm[slot0 + m]; ra = rc / a.e; } else { ra = m; rc = m; }
    }
    sRowA[tid] = ra;
    sRowC[tid] = rc;
  }
  __syncthreads();

  const uint16_t* A = static_cast<const uint16_t*>(a.A);
  const uint16_t* Bm = static_cast<const uint16_t*>(a.Bm) + (size_t)g * a.Ng * a.ldb;

  // global -> register staging: 4 vectors of 8 elements per thread and operand
  const int vrow = tid >> 3;        // 0..31 (+32 per step)
  const int vk = (tid & 7) * 8;     // element offset inside the k tile
  const uint16_t* pa[4];
  const uint16_t* pb[4];
  bool va[4], vb[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = vrow + i * 32;
    const int ra = sRowA[r];
    va[i] = ra >= 0;
    pa[i] = A + (size_t)(va[i] ? ra : 0) * a.lda + vk;
    const int n = n0 + r;
    vb[i] = n < a.Ng;
    pb[i] = Bm + (size_t)(vb[i] ? n : 0) * a.ldb + vk;
  }
  u32x4 ra4[4], rb4[4];
  const u32x4 zero = {0u, 0u, 0u, 0u};
  auto gload = [&](int k0) {
    const bool kin = (k0 + vk) < a.Kdim;  // Kdim % 8 == 0: a vector is fully in or out
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      ra4[i] = (va[i] && kin) ? *reinterpret_cast<const u32x4*>(pa[i] + k0) : zero;
      rb4[i] = (vb[i] && kin) ? *reinterpret_cast<const u32x4*>(pb[i] + k0) : zero;
    }
  };

  const int wave = tid >> 6, lane = tid & 63;
  const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;
  const int fr = lane & 31, fk = (lane >> 5) * 8;
  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  gload(0);
  for (int k0 = 0; k0 < a.Kdim; k0 += BK) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      *reinterpret_cast<u32x4*>(&sA[(vrow + i * 32) * LD + vk]) = ra4[i];
      *reinterpret_cast<u32x4*>(&sB[(vrow + i * 32) * LD + vk]) = rb4[i];
    }
    __syncthreads();
    if (k0 + BK < a.Kdim) gload(k0 + BK);
#pragma unroll
    for (int ks = 0; ks < BK; ks += 16) {
      bf16x8 fa[2], fb[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        fa[i] = *reinterpret_cast<const bf16x8*>(&sA[(wm + i * 32 + fr) * LD + ks + fk]);
        fb[i] = *reinterpret_cast<const bf16x8*>(&sB[(wn + i * 32 + fr) * LD + ks + fk]);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
    }
    __syncthreads();
  }

  // accumulator element r of a 32x32 tile: row (r/4)*8 + (lane/32)*4 + r%4, column lane%32
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int n = n0 + wn + j * 32 + fr;
      if (n >= a.Ng) continue;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int ml = wm + i * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
        const int rc = sRowC[ml];
        if (rc >= 0) a.C[(size_t)rc * a.ldc + n] = acc[i][j][r];
      }
    }
}

// ---------------------------------------------------------------------------------------------
// fp32 inputs: v_mfma_f32_32x32x2_f32 (fp32 products and sums, 157 TFLOP/s at 2.4 GHz where the vector units without packed
// instructions have half of that), tile BM x 64, four waves, k tiles of 32 through two LDS buffers, the loads of the two k
// tiles after the next in registers.
//   BM = 64: waves as 2 x 2, each 32 x 32.
//   BM = 32: waves as 2 (columns) x 2 (halves of every k tile, added through LDS at the end), for problems that would leave
//            compute units with nothing: half the work per tile, and a group of 130 tokens pads to 160 rows instead of 192.
// A fragment read is 16 bytes: four k of one row; instruction j multiplies value j of either operand, so the k are taken in the
// same permuted order in both.  LDS rows of 128 bytes, 16-byte chunk c of row r at chunk c ^ (r & 7).
// The tiles are dealt to the XCDs in eighths, those of a group side by side, so that a group's rows are fetched into one L2.
// Against a vector-unit kernel of 64 x 64 tiles: 1000 tokens x 4 of 32 blocks
// of 256, d 768: 60 -> 32 us; 1000 x 4 of 16 of 256, d 4096: 288 -> 136 (a third of the rate: one barrier per 32 k, and every
// tile's operands out of L2).
// ---------------------------------------------------------------------------------------------
constexpr int kGemmF32BN = 64, kGemmF32BK = 32;

template <int BM>
__global__ __launch_bounds__(256) void gemm_nt_f32_kernel(GemmNTArgs a) {
  constexpr int BN = kGemmF32BN, BK = kGemmF32BK, NL = (BM + BN) * (BK / 4) / 256, WK = BM == 32 ? 2 : 1;
  static_assert(BM == 32 || BM == 64, "");
  __shared__ __attribute__((aligned(16))) float s_buf[2][(BM + BN) * BK];
  __shared__ int sRowA[BM];
  __shared__ int sRowC[BM];

  const int tn = (a.Ng + BN - 1) / BN;
  const int total = (a.perm ? a.tile_off[a.n_groups] : (a.M + BM - 1) / BM) * tn, per = (total + 7) / 8;
  const int tile = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per || tile >= total) return;
  int g, m0, Mg, slot0;
  if (!locate_tile<BM>(a, tile / tn, g, m0, Mg, slot0)) return;
  const int n0 = tile % tn * BN;
  const int tid = threadIdx.x;
  if (tid < BM) {
    const int m = m0 + tid;
    int ra = -1, rc = -1;
    if (m < Mg) {
      if (a.perm) { rc = a.perm[slot0 + m]; ra = rc / a.e; } else { ra = m; rc = m; }
    }
    sRowA[tid] = ra;
    sRowC[tid] = rc;
  }
  __syncthreads();

  const float* A = static_cast<const float*>(a.A);
  const float* Bm = static_cast<const float*>(a.Bm) + (size_t)g * a.Ng * a.ldb;
  // 16-byte words of a k tile: number tid + 256 i is chunk tid % 8 of row tid / 8 + 32 i (A's rows first)
  const int chunk = tid & 7, row0 = tid >> 3;
  const float* src[NL];
  bool valid[NL];
  int at[NL];
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const int r = row0 + 32 * i;
    at[i] = r * BK + ((chunk ^ (r & 7)) << 2);
    if (i < BM / 32) {
      const int ra = sRowA[r];
      valid[i] = ra >= 0;
      src[i] = A + (size_t)(valid[i] ? ra : 0) * a.lda + chunk * 4;
    } else {
      const int n = n0 + r - BM;
      valid[i] = n < a.Ng;
      src[i] = Bm + (size_t)(valid[i] ? n : 0) * a.ldb + chunk * 4;
    }
  }
  struct Stage { f32x4 v[NL]; };
  auto load = [&](int kt, Stage& st) {
    const int k = kt * BK;
    const bool in = k + chunk * 4 < a.Kdim;   // Kdim % 4 == 0
#pragma unroll
    for (int i = 0; i < NL; ++i)
      st.v[i] = in && valid[i] ? *reinterpret_cast<const f32x4*>(src[i] + k) : f32x4{0.f, 0.f, 0.f, 0.f};
  };
  auto put = [&](int buf, const Stage& st) {
#pragma unroll
    for (int i = 0; i < NL; ++i) *reinterpret_cast<f32x4*>(&s_buf[buf][at[i]]) = st.v[i];
  };

  const int wave = tid >> 6, lane = tid & 63, fr = lane & 31, half = lane >> 5;
  const int wm = BM == 32 ? 0 : (wave >> 1) * 32, wn = (wave & 1) * 32, wk = BM == 32 ? wave >> 1 : 0;
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  auto multiply = [&](int buf) {
    const float* pa = &s_buf[buf][(wm + fr) * BK];
    const float* pb = &s_buf[buf][(BM + wn + fr) * BK];
#pragma unroll
    for (int z = 0; z < BK / 8 / WK; ++z) {
      const int c = (((wk * (BK / 8 / WK) + z) * 2 + half) ^ (fr & 7)) << 2;   // rows of a fragment start at multiples of 32
      const f32x4 x = *reinterpret_cast<const f32x4*>(pa + c), y = *reinterpret_cast<const f32x4*>(pb + c);
#pragma unroll
      for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[j], y[j], acc, 0, 0, 0);
    }
  };

  const int nk = (a.Kdim + BK - 1) / BK;
  Stage s0, s1;
  load(0, s0);
  load(1, s1);   // (zeros beyond the end)
  put(0, s0);
  load(2, s0);
  __syncthreads();
  for (int kt = 0; kt < nk; kt += 2) {
    put(1, s1);
    load(kt + 3, s1);
    multiply(0);
    __syncthreads();
    if (kt + 1 >= nk) break;
    put(0, s0);
    load(kt + 4, s0);
    multiply(1);
    __syncthreads();
  }

  // accumulator element r: row (r/4)*8 + (lane/32)*4 + r%4, column lane%32
  if constexpr (WK == 2) {   // (every wave is past its last fragment read)
    f32x4* o = reinterpret_cast<f32x4*>(&s_buf[0][0]) + (wave & 1) * 256 + lane;
    if (wk == 1) {
#pragma unroll
      for (int r = 0; r < 4; ++r) o[r * 64] = f32x4{acc[4 * r], acc[4 * r + 1], acc[4 * r + 2], acc[4 * r + 3]};
    }
    __syncthreads();
    if (wk == 1) return;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const f32x4 v = o[r * 64];
#pragma unroll
      for (int z = 0; z < 4; ++z) acc[4 * r + z] += v[z];
    }
  }
  const int n = n0 + wn + fr;
  if (n >= a.Ng) return;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int rc = sRowC[wm + (r >> 2) * 8 + half * 4 + (r & 3)];
    if (rc >= 0) a.C[(size_t)rc * a.ldc + n] = acc[r];
  }
}

}  // namespace meft
