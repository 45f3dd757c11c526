// Backward weight gradients without floating-point atomics: the (token, neuron) pairs are grouped
// by neuron (counting sort; integer atomics only decide positions, and every group is then put in
// ascending pair order, i.e. ascending token), and the group is summed in that fixed order, in chunks of
// kSegChunk pairs (a wave per chunk and 512 columns; the chunk sums of a long group are added in chunk order):
//   dV[j,:] = sum act * dOut[t,:],  dK[j,:] = sum ds * h[t,:].
// Only touched rows are written.
#pragma once
#include "common.h"

namespace meft {

__global__ void fill_i32_kernel(int32_t* __restrict__ p, size_t n, int32_t v) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// plain streaming copy of n 16-byte words (grid-stride); calibrates bandwidth counters
__global__ __launch_bounds__(256) void probe_copy_kernel(u32x4* __restrict__ dst, const u32x4* __restrict__ src,
                                                         size_t n) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) dst[i] = src[i];
}

// A loop of nothing but matrix instructions: every wave keeps eight independent 32 x 32 accumulators busy with
// v_mfma_f32_32x32x16_bf16 on operands of pseudo-random bits (finite bf16 values; what a matrix core draws depends on
// how many bits toggle).  Gives the rate the matrix cores sustain on this machine: the published peak assumes a
// clock that a chip under this load does not hold.  Each thread stores one float so that the loop is not removed.
__global__ __launch_bounds__(256) void probe_mfma_kernel(float* __restrict__ out, int iters) {
  const uint32_t tid = blockIdx.x * 256u + threadIdx.x;
  uint32_t x = tid * 2654435761u + 12345u;
  auto next = [&]() {   // two bf16 values with exponents 0x3F/0x40: magnitudes between 0.5 and 4, random signs
    x = x * 1664525u + 1013904223u;
    return (x & 0x80FF80FFu) | 0x3F003F00u;
  };
  bf16x8 a[2], b[4];
#pragma unroll
  for (int i = 0; i < 2; ++i) a[i] = __builtin_bit_cast(bf16x8, u32x4{next(), next(), next(), next()});
#pragma unroll
  for (int j = 0; j < 4; ++j) b[j] = __builtin_bit_cast(bf16x8, u32x4{next(), next(), next(), next()});
  f32x16 acc[2][4];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
  }
  float sum = 0.f;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) sum += acc[i][j][r];
  out[tid] = sum;
}

// block id of every (token, neuron) pair (ids clamped into range)
__global__ void blocks_of_pairs_kernel(const int32_t* __restrict__ idx, int P, int N, int bs,
                                       int32_t* __restrict__ blk) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p < P) blk[p] = clampi(idx[p], 0, N - 1) / bs;
}

// copies the rows listed in touched[0 .. *n_touched) from a device matrix to the same rows of a matrix in
// pinned host memory (the device writes over the host link); one workgroup per listed row, `vec` 16-byte
// words per row
__global__ __launch_bounds__(256) void rows_to_host_kernel(const int32_t* __restrict__ touched,
                                                           const int32_t* __restrict__ n_touched,
                                                           const u32x4* __restrict__ src, u32x4* __restrict__ dst,
                                                           int vec) {
  const int u = blockIdx.x;
  if (u >= *n_touched) return;
  const size_t row = (size_t)touched[u] * vec;
  for (int i = threadIdx.x; i < vec; i += 256) dst[row + i] = src[row + i];
}

// cnt[j] += 1 for every pair; pos[p] = the pair's place in its neuron's segment, in the order of arrival
__global__ void pair_count_kernel(const int32_t* __restrict__ idx, int P, int N, int32_t* __restrict__ cnt,
                                  int32_t* __restrict__ pos) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p < P) pos[p] = atomicAdd(&cnt[clampi(idx[p], 0, N - 1)], 1);
}

// A neuron's pairs are summed in chunks of kSegChunk consecutive pairs, so that a neuron that very many tokens selected does
// not leave one wave with all of its pairs.
constexpr int kSegChunk = 256;

// What one chunk is: neuron, first pair in the grouped list, number of pairs, and its row in the buffer of partial sums
// (-1: the only chunk of its neuron, which is written directly).
struct SegWork {
  int j, off, len, part;
};

// Per touched neuron u (ascending id): touched[u], and its chunks in work[]; per neuron of more than one chunk an entry
// (neuron, first row of partial sums, chunks) in multi[]; seg_off = exclusive scan of cnt.  totals = {touched, chunks,
// neurons of more than one chunk}.  A workgroup of 256 threads takes kScanChunk counters and adds up the ones before them
// itself, out of L2 (one workgroup for all of them took 119 us at 65536 neurons, this 16 us), or, beyond kScanSelfMax
// counters, takes the sums that pair_sums_kernel left.
constexpr int kScanChunk = 2048, kScanSelfMax = 1 << 17;
struct PairSums {
  int c, f, wk, mu, mn;   // pairs, touched neurons, chunks, chunks of neurons with several, such neurons
  __device__ __forceinline__ void add(int v) {
    const int ch = (v + kSegChunk - 1) / kSegChunk;
    c += v; f += v > 0; wk += ch; mu += ch > 1 ? ch : 0; mn += ch > 1 ? 1 : 0;
  }
};

// sums over a workgroup of 256 threads, in every thread (s: 5 x 4 ints)
__device__ __forceinline__ PairSums pair_sums_all(PairSums x, int (*s)[4]) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int v[5] = {x.c, x.f, x.wk, x.mu, x.mn};
  int r[5];
#pragma unroll
  for (int z = 0; z < 5; ++z) {
    const int incl = wave_incl_scan(v[z]);
    if (lane == 63) s[z][w] = incl;
  }
  __syncthreads();
#pragma unroll
  for (int z = 0; z < 5; ++z) r[z] = s[z][0] + s[z][1] + s[z][2] + s[z][3];
  __syncthreads();
  return PairSums{r[0], r[1], r[2], r[3], r[4]};
}

__global__ __launch_bounds__(256) void pair_sums_kernel(const int32_t* __restrict__ cnt, int N, PairSums* __restrict__ sums) {
  __shared__ int s[5][4];
  PairSums x{0, 0, 0, 0, 0};
  const int j0 = blockIdx.x * kScanChunk + threadIdx.x * 8;
#pragma unroll
  for (int z = 0; z < 8; ++z)
    if (j0 + z < N) x.add(cnt[j0 + z]);
  x = pair_sums_all(x, s);
  if (threadIdx.x == 0) sums[blockIdx.x] = x;
}

__global__ __launch_bounds__(256) void pair_scan_kernel(const int32_t* __restrict__ cnt, int N,
                                                        const PairSums* __restrict__ sums,
                                                        int32_t* __restrict__ seg_off, int32_t* __restrict__ touched,
                                                        int32_t* __restrict__ n_touched, SegWork* __restrict__ work,
                                                        int4* __restrict__ multi, int32_t* __restrict__ totals) {
  __shared__ int s[5][4];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, chunk = blockIdx.x;
  PairSums before{0, 0, 0, 0, 0};
  if (sums != nullptr) {
    for (int c = tid; c < chunk; c += 256) {
      const PairSums y = sums[c];
      before.c += y.c; before.f += y.f; before.wk += y.wk; before.mu += y.mu; before.mn += y.mn;
    }
  } else {
    const i32x4* c4 = reinterpret_cast<const i32x4*>(cnt);
#pragma unroll 4
    for (int c = tid; c < chunk * (kScanChunk / 4); c += 256) {
      const i32x4 v = c4[c];
      before.add(v.x); before.add(v.y); before.add(v.z); before.add(v.w);
    }
  }
  before = pair_sums_all(before, s);
  const int j0 = chunk * kScanChunk + tid * 8;
  int v[8];
  PairSums mine{0, 0, 0, 0, 0};
#pragma unroll
  for (int z = 0; z < 8; ++z) {
    v[z] = j0 + z < N ? cnt[j0 + z] : 0;
    mine.add(v[z]);
  }
  // exclusive prefix of the thread's sums inside the workgroup
  const int m[5] = {mine.c, mine.f, mine.wk, mine.mu, mine.mn};
  int ex[5];
#pragma unroll
  for (int z = 0; z < 5; ++z) {
    const int incl = wave_incl_scan(m[z]);
    if (lane == 63) s[z][w] = incl;
    ex[z] = incl - m[z];
  }
  __syncthreads();
#pragma unroll
  for (int z = 0; z < 5; ++z)
    for (int i = 0; i < w; ++i) ex[z] += s[z][i];
  int off = before.c + ex[0], nt = before.f + ex[1], wo = before.wk + ex[2], mo = before.mu + ex[3], mn = before.mn + ex[4];
#pragma unroll
  for (int z = 0; z < 8; ++z) {
    if (j0 + z < N) seg_off[j0 + z] = off;
    if (v[z] > 0) {
      const int ch = (v[z] + kSegChunk - 1) / kSegChunk;
      touched[nt++] = j0 + z;
      if (ch > 1) multi[mn++] = make_int4(j0 + z, mo, ch, 0);
      for (int c = 0; c < ch; ++c)
        work[wo++] = SegWork{j0 + z, off + c * kSegChunk, min(v[z] - c * kSegChunk, kSegChunk), ch > 1 ? mo++ : -1};
    }
    off += v[z];
  }
  if (chunk == (int)gridDim.x - 1 && tid == 255) {
    seg_off[N] = off;
    *n_touched = nt;
    totals[0] = nt; totals[1] = wo; totals[2] = mn;
  }
}

// unordered placement of the pairs into their neuron's segment
__global__ void pair_fill_kernel(const int32_t* __restrict__ idx, int P, int N,
                                 const int32_t* __restrict__ seg_off, const int32_t* __restrict__ pos,
                                 int32_t* __restrict__ pair_list) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= P) return;
  const int j = clampi(idx[p], 0, N - 1);
  pair_list[seg_off[j] + pos[p]] = p;
}

// Puts the segments of more than kSegChunk pairs in ascending pair order (pair ids are distinct); the shorter ones are put
// in order by the kernel that sums them.  Up to kBitonicMax: a bitonic sort in LDS (a neuron that thousands of tokens
// selected would cost L^2 comparisons otherwise).  Beyond that (more tokens than kBitonicMax selected one neuron): ranks
// counted against global memory, slow but never wrong.
__global__ __launch_bounds__(256) void seg_sort_kernel(const int4* __restrict__ multi, const int32_t* __restrict__ totals,
                                                       const int32_t* __restrict__ seg_off,
                                                       const int32_t* __restrict__ pair_list,
                                                       int32_t* __restrict__ pair_sorted) {
  constexpr int kBitonicMax = 8192;
  __shared__ int32_t s_p[kBitonicMax];
  for (int u = blockIdx.x; u < totals[2]; u += gridDim.x) {
    const int j = multi[u].x;
    const int o = seg_off[j], L = seg_off[j + 1] - o;
    const int32_t* src = pair_list + o;
    if (L <= kBitonicMax) {
      int n = 512;
      while (n < L) n <<= 1;
      for (int i = threadIdx.x; i < n; i += 256) s_p[i] = i < L ? src[i] : 0x7FFFFFFF;   // padding sorts to the end
      __syncthreads();
      for (int size = 2; size <= n; size <<= 1)
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
          for (int i = threadIdx.x; i < n / 2; i += 256) {
            const int lo = ((i / stride) * stride * 2) + (i % stride), hi = lo + stride;
            const bool up = (lo & size) == 0;   // ascending half of this merge
            const int a = s_p[lo], b = s_p[hi];
            if ((a > b) == up) { s_p[lo] = b; s_p[hi] = a; }
          }
          __syncthreads();
        }
      for (int i = threadIdx.x; i < L; i += 256) pair_sorted[o + i] = s_p[i];
      __syncthreads();
    } else {
      for (int i = threadIdx.x; i < L; i += 256) {
        const int v = src[i];
        int r = 0;
        for (int z = 0; z < L; ++z) r += src[z] < v;
        pair_sorted[o + r] = v;
      }
    }
  }
}

// One chunk of a touched neuron's pairs, summed in ascending pair order (which is ascending token order): dV[j,:] = sum
// act * dOut[t,:], dK[j,:] = sum ds * h[t,:].  A wave takes (chunk, 512 columns), a workgroup four chunks of the same
// columns.  The columns are the slow launch index (y): while a slice of 512 columns is worked through, the slices of h and
// dOut (2 MB each at 2048 bf16 tokens) stay in the L2 of every XCD, and the row reads, of which there is one pair per
// (token, neuron) pair, no longer go to memory.  A neuron of one chunk gets its rows written here; the chunks of a longer
// segment leave their fp32 sums in `part` ([chunk][dV | dK][d]), which seg_finish_kernel adds in chunk order.
// 2048 tokens x 256 pairs, d 4096, bf16, 65536 neurons (8.6 GB of rows, 1.1 GB written): 1148 + 73 us (rows of a
// workgroup, segments sorted in a launch of their own) -> 577 us, 15 TB/s of rows out of L2.
template <typename T>
__global__ __launch_bounds__(256) void seg_reduce_kernel(const SegWork* __restrict__ work, const int32_t* __restrict__ totals,
                                                         const int32_t* __restrict__ pair_list,
                                                         const int32_t* __restrict__ pair_sorted,
                                                         const float* __restrict__ act, const float* __restrict__ ds,
                                                         const T* __restrict__ h, const T* __restrict__ dOut, int d, int k,
                                                         T* __restrict__ dK, T* __restrict__ dV, float* __restrict__ part) {
  __shared__ int s_p[4][kSegChunk];
  __shared__ float2 s_c[4][kSegChunk];   // act, ds
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int slice = blockIdx.y, wk = blockIdx.x * 4 + wave;
  if (wk >= totals[1]) return;   // (no workgroup barrier below: every wave keeps to its own part of LDS)
  const SegWork x = work[wk];
  int* sp = s_p[wave];
  float2* scf = s_c[wave];
  if (x.part < 0) {
    // rank of every pair among the chunk's (at most four per lane)
    int v[kSegChunk / 64], r[kSegChunk / 64];
#pragma unroll
    for (int z = 0; z < kSegChunk / 64; ++z) {
      v[z] = z * 64 + lane < x.len ? pair_list[x.off + z * 64 + lane] : 0x7FFFFFFF;
      r[z] = 0;
      sp[z * 64 + lane] = v[z];
    }
    wave_lds_fence();
    for (int i = 0; i < x.len; ++i) {
      const int y = sp[i];
#pragma unroll
      for (int z = 0; z < kSegChunk / 64; ++z) r[z] += y < v[z] ? 1 : 0;
    }
    wave_lds_fence();
#pragma unroll
    for (int z = 0; z < kSegChunk / 64; ++z)
      if (z * 64 + lane < x.len) sp[r[z]] = v[z];
  } else {
#pragma unroll
    for (int z = 0; z < kSegChunk / 64; ++z)
      if (z * 64 + lane < x.len) sp[z * 64 + lane] = pair_sorted[x.off + z * 64 + lane];
  }
  wave_lds_fence();
  for (int i = lane; i < x.len; i += 64) {
    const int p = sp[i];
    scf[i] = make_float2(act[p], ds[p]);
    sp[i] = p / k;
  }
  wave_lds_fence();
  const int col = slice * 512 + lane * 8;
  if (col >= d) return;
  float aK[8], aV[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) { aK[c] = 0.f; aV[c] = 0.f; }
  constexpr int U = 4, W = Vec8<T>::kBytes / 16;
  for (int q = 0; q < x.len; q += U) {
    u32x4 xg[U][W], xh[U][W];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const size_t at = (size_t)sp[min(q + u, x.len - 1)] * d + col;
#pragma unroll
      for (int w = 0; w < W; ++w) {
        xg[u][w] = reinterpret_cast<const u32x4*>(dOut + at)[w];
        xh[u][w] = reinterpret_cast<const u32x4*>(h + at)[w];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (q + u < x.len) {
        const float2 cf = scf[q + u];
        float g[8], hh[8];
        Vec8<T>::load(reinterpret_cast<const T*>(&xg[u][0]), g);
        Vec8<T>::load(reinterpret_cast<const T*>(&xh[u][0]), hh);
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          aV[c] = fmaf(cf.x, g[c], aV[c]);
          aK[c] = fmaf(cf.y, hh[c], aK[c]);
        }
      }
    }
  }
  if (x.part < 0) {
    Vec8<T>::store(dV + (size_t)x.j * d + col, aV);
    Vec8<T>::store(dK + (size_t)x.j * d + col, aK);
  } else {
    float* pv = part + (size_t)x.part * 2 * d + col;
    Vec8<float>::store(pv, aV);
    Vec8<float>::store(pv + d, aK);
  }
}

// The rows of the touched neurons of more than one chunk: their chunks' partial sums added in chunk order.
template <typename T>
__global__ __launch_bounds__(256) void seg_finish_kernel(const int4* __restrict__ multi, const int32_t* __restrict__ totals,
                                                         const float* __restrict__ part, int d, T* __restrict__ dK,
                                                         T* __restrict__ dV) {
  for (int u = blockIdx.x; u < totals[2]; u += gridDim.x) {
    const int4 m = multi[u];
    const float* pv = part + (size_t)m.y * 2 * d;
    for (int col = threadIdx.x * 8; col < d; col += 256 * 8) {
      float aK[8], aV[8];
#pragma unroll
      for (int c = 0; c < 8; ++c) { aK[c] = 0.f; aV[c] = 0.f; }
      for (int c = 0; c < m.z; ++c) {
        float xv[8], xk[8];
        Vec8<float>::load(pv + (size_t)c * 2 * d + col, xv);
        Vec8<float>::load(pv + (size_t)c * 2 * d + d + col, xk);
#pragma unroll
        for (int cc = 0; cc < 8; ++cc) { aV[cc] += xv[cc]; aK[cc] += xk[cc]; }
      }
      Vec8<T>::store(dV + (size_t)m.x * d + col, aV);
      Vec8<T>::store(dK + (size_t)m.x * d + col, aK);
    }
  }
}

}  // namespace meft
