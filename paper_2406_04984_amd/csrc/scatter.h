// Backward of the per-pair path without floating-point atomics: the (token, neuron) pairs are grouped by neuron (counting
// sort; integer atomics only decide positions, and every group is then put in ascending pair order, i.e. ascending token),
// and the group is worked through in that fixed order, in chunks of kSegChunk pairs (a wave per chunk and 1 KB of columns;
// the chunk sums of a long group are added in chunk order):
//   dV[j,:] = sum act * dOut[t,:],  ds = act > 0 ? dOut[t,:] . V[j,:] : 0,  dK[j,:] = sum ds * h[t,:].
// Only touched rows are written.  A token's dh, the sum of ds * K[j,:] over its pairs, follows in gather.h.
#pragma once
#include <type_traits>

#include "common.h"
#include "select.h"

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
// neurons of more than one chunk}.  A workgroup of 1024 threads takes kScanChunk counters and adds up the ones before them
// itself, out of L2 (65536 neurons: 119 us by one workgroup for all of them, 15 us so, 9 us with eight loads of a thread together,
// short sums where no counter is of more than a chunk, and one pass over the waves' sums), or, beyond
// kScanSelfMax counters, takes the sums that pair_sums_kernel left.
constexpr int kScanChunk = 2048, kScanSelfMax = 1 << 17, kScanThreads = 1024, kScanPer = kScanChunk / kScanThreads;
struct PairSums {
  int c, f, wk, mu, mn;   // pairs, touched neurons, chunks, chunks of neurons with several, such neurons
  __device__ __forceinline__ void add(int v) {
    const int ch = (v + kSegChunk - 1) / kSegChunk;
    c += v; f += v > 0; wk += ch; mu += ch > 1 ? ch : 0; mn += ch > 1 ? 1 : 0;
  }
  // four counters: mostly, none is of more than a chunk
  __device__ __forceinline__ void add4(i32x4 v) {
    if (max(max(v.x, v.y), max(v.z, v.w)) > kSegChunk) {
      add(v.x); add(v.y); add(v.z); add(v.w);
      return;
    }
    const int n = (v.x > 0) + (v.y > 0) + (v.z > 0) + (v.w > 0);
    c += v.x + v.y + v.z + v.w; f += n; wk += n;
  }
};

__global__ __launch_bounds__(kScanThreads) void pair_sums_kernel(const int32_t* __restrict__ cnt, int N, PairSums* __restrict__ sums) {
  __shared__ int s[kScanThreads / 64][5];
  PairSums x{0, 0, 0, 0, 0};
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, j0 = blockIdx.x * kScanChunk + threadIdx.x * kScanPer;
#pragma unroll
  for (int z = 0; z < kScanPer; ++z)
    if (j0 + z < N) x.add(cnt[j0 + z]);
  const int v[5] = {x.c, x.f, x.wk, x.mu, x.mn};
#pragma unroll
  for (int z = 0; z < 5; ++z) {
    const int incl = wave_incl_scan(v[z]);
    if (lane == 63) s[w][z] = incl;
  }
  __syncthreads();
  if (threadIdx.x < 5) {
    int r = 0;
#pragma unroll
    for (int i = 0; i < kScanThreads / 64; ++i) r += s[i][threadIdx.x];
    (&sums[blockIdx.x].c)[threadIdx.x] = r;
  }
}

__global__ __launch_bounds__(kScanThreads) void pair_scan_kernel(const int32_t* __restrict__ cnt, int N,
                                                        const PairSums* __restrict__ sums,
                                                        int32_t* __restrict__ seg_off, int32_t* __restrict__ touched,
                                                        int32_t* __restrict__ n_touched, SegWork* __restrict__ work,
                                                        int4* __restrict__ multi, int32_t* __restrict__ totals) {
  constexpr int kWaves = kScanThreads / 64;
  __shared__ int s_before[5][kWaves], s_mine[5][kWaves];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), chunk = blockIdx.x;
  const int j0 = chunk * kScanChunk + tid * kScanPer;
  int v[kScanPer];
  PairSums mine{0, 0, 0, 0, 0};
#pragma unroll
  for (int z = 0; z < kScanPer; ++z) v[z] = j0 + z < N ? cnt[j0 + z] : 0;
  PairSums before{0, 0, 0, 0, 0};
  if (sums != nullptr) {
    for (int c = tid; c < chunk; c += kScanThreads) {
      const PairSums y = sums[c];
      before.c += y.c; before.f += y.f; before.wk += y.wk; before.mu += y.mu; before.mn += y.mn;
    }
  } else {
    const i32x4* c4 = reinterpret_cast<const i32x4*>(cnt);
    const int n = chunk * (kScanChunk / 4);
    for (int c = tid; c < n; c += 8 * kScanThreads) {   // (eight loads on their way together)
      i32x4 x[8];
#pragma unroll
      for (int z = 0; z < 8; ++z) x[z] = c4[min(c + kScanThreads * z, n - 1)];
#pragma unroll
      for (int z = 0; z < 8; ++z)
        if (c + kScanThreads * z < n) before.add4(x[z]);
    }
  }
#pragma unroll
  for (int z = 0; z < kScanPer; ++z) mine.add(v[z]);
  // per wave, then over the waves (a lane each): the sums before the workgroup and the prefix inside it.  Short chains of
  // instructions: this is what a workgroup with few counters before it takes.
  const int b[5] = {before.c, before.f, before.wk, before.mu, before.mn}, m[5] = {mine.c, mine.f, mine.wk, mine.mu, mine.mn};
  int ex[5];
#pragma unroll
  for (int z = 0; z < 5; ++z) {
    const int all = wave_incl_scan(b[z]), incl = wave_incl_scan(m[z]);
    if (lane == 63) { s_before[z][w] = all; s_mine[z][w] = incl; }
    ex[z] = incl - m[z];
  }
  __syncthreads();
#pragma unroll
  for (int z = 0; z < 5; ++z) {
    const int waves = wave_incl_scan(lane < kWaves ? s_before[z][lane % kWaves] : lane < 2 * kWaves && lane - kWaves < w ? s_mine[z][lane % kWaves] : 0);
    ex[z] += __builtin_amdgcn_readlane(waves, 63);
  }
  int off = ex[0], nt = ex[1], wo = ex[2], mo = ex[3], mn = ex[4];
#pragma unroll
  for (int z = 0; z < kScanPer; ++z) {
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
  if (chunk == (int)gridDim.x - 1 && tid == kScanThreads - 1) {
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

// Puts one segment of L > kSegChunk pairs in ascending order, by a workgroup of NT threads: up to kBitonicMax by a bitonic sort
// in LDS (a neuron that thousands of tokens selected would cost L^2 comparisons otherwise), beyond that (more tokens than
// kBitonicMax selected one neuron) by ranks counted against the segment, which comes through LDS kBitonicMax pairs at a time: slow
// but never wrong (65536 tokens x 16 pairs of 64 neurons: the whole backward 38.6 ms with the ranks counted against memory,
// 8.2 ms so).  put(i, p): pair p is the i-th.
constexpr int kBitonicMax = 8192;
template <int NT, class Put>
__device__ __forceinline__ void sort_long_segment(const int32_t* src, int L, int32_t* s_p, Put&& put) {
  if (L <= kBitonicMax) {
    int n = 512;
    while (n < L) n <<= 1;
    for (int i = threadIdx.x; i < n; i += NT) s_p[i] = i < L ? src[i] : 0x7FFFFFFF;   // padding sorts to the end
    __syncthreads();
    for (int size = 2; size <= n; size <<= 1)
      for (int stride = size >> 1; stride > 0; stride >>= 1) {
        for (int i = threadIdx.x; i < n / 2; i += NT) {
          const int lo = ((i / stride) * stride * 2) + (i % stride), hi = lo + stride;
          const bool up = (lo & size) == 0;   // ascending half of this merge
          const int a = s_p[lo], b = s_p[hi];
          if ((a > b) == up) { s_p[lo] = b; s_p[hi] = a; }
        }
        __syncthreads();
      }
    for (int i = threadIdx.x; i < L; i += NT) put(i, s_p[i]);
    __syncthreads();
    return;
  }
  constexpr int kOwn = 8;   // pairs a thread ranks at a time
  for (int i0 = threadIdx.x; i0 - (int)threadIdx.x < L; i0 += NT * kOwn) {
    int v[kOwn], r[kOwn];
#pragma unroll
    for (int z = 0; z < kOwn; ++z) { v[z] = i0 + NT * z < L ? src[i0 + NT * z] : 0; r[z] = 0; }
    for (int b = 0; b < L; b += kBitonicMax) {
      const int n = min(kBitonicMax, L - b);
      __syncthreads();
      for (int i = threadIdx.x; i < (n + 3) / 4 * 4; i += NT) s_p[i] = i < n ? src[b + i] : 0x7FFFFFFF;
      __syncthreads();
      for (int i = 0; i < n; i += 4) {
        const i32x4 y = *reinterpret_cast<const i32x4*>(&s_p[i]);
#pragma unroll
        for (int z = 0; z < kOwn; ++z) r[z] += (y.x < v[z]) + (y.y < v[z]) + (y.z < v[z]) + (y.w < v[z]);
      }
    }
#pragma unroll
    for (int z = 0; z < kOwn; ++z)
      if (i0 + NT * z < L) put(r[z], v[z]);
  }
  __syncthreads();
}

// Puts every segment in ascending pair order (pair ids are distinct) and notes (token, activation) of its pairs beside it, so
// that the kernels that sum a segment, once per 1 KB of columns, find both with one coalesced read.  Workgroups 0 .. n_multi - 1
// take the segments of more than kSegChunk pairs; the others the pairs of the remaining segments, a thread
// each, which counts the pair's rank among the at most kSegChunk of its neuron (a wave per segment: 18 instead of 6.5 us
// at 64000 pairs of 41000 neurons).
__global__ __launch_bounds__(256) void seg_sort_kernel(const int4* __restrict__ multi,
                                                       const int32_t* __restrict__ totals,
                                                       const int32_t* __restrict__ seg_off,
                                                       const int32_t* __restrict__ pair_list,
                                                       const int32_t* __restrict__ idx, const float* __restrict__ act,
                                                       int P, int N, int k, int n_multi, int32_t* __restrict__ pair_sorted,
                                                       int2* __restrict__ seg) {
  __shared__ __attribute__((aligned(16))) int32_t s_p[kBitonicMax];
  auto put = [&](int at, int p) {
    pair_sorted[at] = p;
    seg[at] = make_int2(p / k, __float_as_int(act[p]));
  };
  if ((int)blockIdx.x < n_multi) {
    for (int u = blockIdx.x; u < totals[2]; u += n_multi) {
      const int j = multi[u].x;
      const int o = seg_off[j];
      sort_long_segment<256>(pair_list + o, seg_off[j + 1] - o, s_p, [&](int i, int p) { put(o + i, p); });
    }
    return;
  }
  const int i = ((int)blockIdx.x - n_multi) * 256 + (int)threadIdx.x;
  if (i >= P) return;
  const int p = pair_list[i], j = clampi(idx[p], 0, N - 1);
  const int o = seg_off[j], L = seg_off[j + 1] - o;
  if (L > kSegChunk) return;
  int r = 0;
#pragma unroll 4
  for (int z = 0; z < L; ++z) r += pair_list[o + z] < p ? 1 : 0;
  put(o + r, p);
}

// All of the above in one launch, for up to kPairOneP pairs.  Every workgroup counts all pairs by bucket (2^shift consecutive
// neurons, so that kPairOneBuckets cover them all) in LDS; bucket b belongs to workgroup b % kPairOneWgs, which lists its pairs
// and puts them in order of (neuron, pair).  Nobody counts the touched neurons before a bucket, so the work entries are not
// compacted: entry i is about the i-th pair in order, and holds a chunk where that is the chunk's first pair (len 0: none).
// first[i] = neuron where the pair is its neuron's first (~neuron where the neuron has more than one chunk, which are then
// described in multi[i / kSegChunk]), kNotFirst elsewhere: pair_lists_body makes the lists out of that.
// The five launches that this replaces depend on each other and take 2 to 12 us each, however few the pairs; this one takes 5 at 8192
// pairs.  Backward, five launches / one, us: 512 tokens x 16 pairs, d 256 bf16, 20480 neurons 33.5 / 22.5, 262144 neurons 36.8 /
// 23.8; 250 x 64, d 784 fp32, 65536 neurons 70.9 / 61.2.  With more pairs the looking through all of them by every workgroup
// costs what the launches do: 24000 pairs of 20000 neurons, d 256 fp32 40.0 / 39.7, d 512 bf16 41.4 / 41.7.
constexpr int kPairBits = 15, kPairOneBatch = 20, kPairOneP = kPairOneBatch * kScanThreads, kPairOneBuckets = 4096, kPairOneWgs = 128;
constexpr int kPairOneOwn = kPairOneBuckets / kPairOneWgs, kNotFirst = INT32_MIN;

// A thread keeps kBatch pairs: 8 where they are enough, kPairOneBatch otherwise.
template <int kBatch>
__global__ __launch_bounds__(kScanThreads) void pair_one_kernel(const int32_t* __restrict__ idx, const float* __restrict__ act, int P,
                                                       int N, int k, int shift, SegWork* __restrict__ work,
                                                       int4* __restrict__ multi, int32_t* __restrict__ first,
                                                       int32_t* __restrict__ pair_sorted, int2* __restrict__ seg) {
  constexpr int kPer = kPairOneBuckets / kScanThreads;   // consecutive counters of a thread
  constexpr uint32_t kPairMask = (1u << kPairBits) - 1;
  static_assert(kPer == 4 && kPairOneOwn <= 32, "");
  extern __shared__ uint32_t s_keys[];   // [P]: the workgroup's pairs, bucket by bucket: (neuron - bucket's first) << kPairBits | pair
  __shared__ __attribute__((aligned(16))) int32_t s_cnt[kPairOneBuckets + 4];   // pairs of the bucket, then its first place
  __shared__ int32_t s_off[kPairOneOwn + 1], s_at[kPairOneOwn], s_w[kScanThreads / 64];   // own buckets: where in s_keys
  const int tid = threadIdx.x, wg = blockIdx.x;
  int jp[kBatch];   // neurons of the pairs tid + kScanThreads * z
#pragma unroll
  for (int z = 0; z < kBatch; ++z) jp[z] = idx[min(tid + kScanThreads * z, P - 1)];
  auto pairs = [&](auto&& f) {   // f(pair, neuron) for every pair
#pragma unroll
    for (int z = 0; z < kBatch; ++z)
      if (tid + kScanThreads * z < P) f(tid + kScanThreads * z, clampi(jp[z], 0, N - 1));
  };
  i32x4* cnt4 = reinterpret_cast<i32x4*>(s_cnt) + tid;
  *cnt4 = i32x4{0, 0, 0, 0};
  __syncthreads();
  pairs([&](int, int j) { atomicAdd(&s_cnt[j >> shift], 1); });
  __syncthreads();
  const i32x4 v = *cnt4;
  int all;
  const int off = block_excl_scan_1024(v.x + v.y + v.z + v.w, s_w, all);   // (its barriers part the reads from the writes)
  *cnt4 = i32x4{off, off + v.x, off + v.x + v.y, off + v.x + v.y + v.z};
  if (tid == 0) s_cnt[kPairOneBuckets] = all;
  __syncthreads();
  if (tid < 64) {
    const int b = min(tid, kPairOneOwn - 1) * kPairOneWgs + wg, len = tid < kPairOneOwn ? s_cnt[b + 1] - s_cnt[b] : 0;
    const int incl = wave_incl_scan(len);
    if (tid < kPairOneOwn) { s_off[tid] = s_at[tid] = incl - len; s_off[tid + 1] = incl; }   // (the same value from either writer)
  }
  __syncthreads();
  pairs([&](int p, int j) {
    const int b = j >> shift;
    if (b % kPairOneWgs == wg) s_keys[atomicAdd(&s_at[b / kPairOneWgs], 1)] = (uint32_t)(j - (b << shift)) << kPairBits | (uint32_t)p;
  });
  __syncthreads();
  // pair `key` of own bucket m is the r-th of the bucket, which has `before` pairs of lesser neurons, `upto` up to its neuron
  auto put = [&](int m, uint32_t key, int r, int before, int upto) {
    const int b = m * kPairOneWgs + wg, p = (int)(key & kPairMask), j = (b << shift) + (int)(key >> kPairBits);
    const int i = s_cnt[b] + r, e = r - before, L = upto - before;
    // (rows of partial sums: a neuron of L > 256 pairs has at most L / 128 chunks)
    const int row = L > kSegChunk ? (i - e) / (kSegChunk / 2) : -1;
    pair_sorted[i] = p;
    seg[i] = make_int2(p / k, __float_as_int(act[p]));
    first[i] = e > 0 ? kNotFirst : row < 0 ? j : ~j;
    work[i] = SegWork{j, i, e % kSegChunk == 0 ? min(L - e, kSegChunk) : 0, row < 0 ? -1 : row + e / kSegChunk};
    if (e == 0 && row >= 0) multi[i / kSegChunk] = make_int4(j, row, (L + kSegChunk - 1) / kSegChunk, 0);
  };
  // a thread per pair of the workgroup counts its rank in buckets of a chunk or less
  for (int x = tid; x < s_off[kPairOneOwn]; x += kScanThreads) {
    int m = 0;
#pragma unroll
    for (int z = kPairOneOwn / 2; z > 0; z >>= 1) m += s_off[m + z] <= x ? z : 0;
    const int o = s_off[m], L = s_off[m + 1] - o;
    if (L > kSegChunk) continue;
    const uint32_t key = s_keys[x], from = key & ~kPairMask, to = key | kPairMask;
    int r = 0, before = 0, upto = 0;
#pragma unroll 4
    for (int y = 0; y < L; ++y) {
      const uint32_t other = s_keys[o + y];
      r += other < key ? 1 : 0;
      before += other < from ? 1 : 0;
      upto += other <= to ? 1 : 0;
    }
    put(m, key, r, before, upto);
  }
  __syncthreads();
  // larger ones are sorted where they are: a bitonic network whose exchanges all put the lesser key first, so that places
  // beyond the end can be left out
  for (int m = 0; m < kPairOneOwn; ++m) {
    const int o = s_off[m], L = s_off[m + 1] - o;
    if (L <= kSegChunk) continue;
    uint32_t* a = s_keys + o;
    auto order = [&](int lo, int hi) {
      if (hi < L) {
        const uint32_t x = a[lo], y = a[hi];
        if (x > y) { a[lo] = y; a[hi] = x; }
      }
    };
    int lgn = 1;
    while ((1 << lgn) < L) ++lgn;
    for (int lg = 1; lg <= lgn; ++lg) {
      for (int i = tid; i < 1 << (lgn - 1); i += kScanThreads) {   // i-th pair of places: mirrored in pieces of 2^lg
        const int base = (i >> (lg - 1)) << lg, x = i & ((1 << (lg - 1)) - 1);
        order(base + x, base + (1 << lg) - 1 - x);
      }
      __syncthreads();
      for (int st = lg - 2; st >= 0; --st) {
        for (int i = tid; i < 1 << (lgn - 1); i += kScanThreads) {
          const int lo = (i >> st) << (st + 1) | (i & ((1 << st) - 1));
          order(lo, lo + (1 << st));
        }
        __syncthreads();
      }
    }
    auto below = [&](uint32_t x) {   // keys less than x
      int lo = 0, hi = L;
      while (lo < hi) {
        const int h = (lo + hi) >> 1;
        if (a[h] < x) lo = h + 1; else hi = h;
      }
      return lo;
    };
    for (int r = tid; r < L; r += kScanThreads) {
      const uint32_t key = a[r], to = key | kPairMask;
      put(m, key, r, below(key & ~kPairMask), to == 0xFFFFFFFFu ? L : below(to + 1));
    }
  }
}

// The lists that pair_one_kernel's entries stand for: touched neurons, ascending, and the neurons of more than one chunk.  Executed by
// one workgroup of 256 threads, a thread for kPairListPer consecutive entries at a time.
constexpr int kPairListPer = 32;
struct PairLists {
  const int32_t* first;   // nullptr: the lists are there
  int n_pairs;
  int32_t *touched, *n_touched;
  int4* multi;
  int32_t* totals;
};
__device__ __forceinline__ void pair_lists_body(const PairLists& l) {
  constexpr int kWindows = kPairOneP / kSegChunk;   // each holds the first pair of at most one neuron of more than one chunk
  __shared__ int s_w[4], s_long[kWindows];
  static_assert(kWindows <= 256, "");
  const int tid = threadIdx.x, P = l.n_pairs;
  if (tid < kWindows) s_long[tid] = 0;
  __syncthreads();
  int total = 0;
#pragma unroll 1
  for (int t0 = 0; t0 < P; t0 += 256 * kPairListPer) {
    const int i0 = t0 + tid * kPairListPer;
    int32_t v[kPairListPer];
    int n = 0;
#pragma unroll
    for (int z = 0; z < kPairListPer; z += 4) {   // (arrays of the workspace are whole 256-byte pieces)
      const i32x4 x = *reinterpret_cast<const i32x4*>(l.first + min(i0 + z, (P - 1) & ~3));
#pragma unroll
      for (int y = 0; y < 4; ++y) {
        v[z + y] = i0 + z + y < P ? x[y] : kNotFirst;
        n += v[z + y] != kNotFirst ? 1 : 0;
        if (v[z + y] < 0 && v[z + y] != kNotFirst) s_long[(i0 + z + y) / kSegChunk] = 1;
      }
    }
    int all, at = total + block_excl_scan_256(n, s_w, all);
#pragma unroll
    for (int z = 0; z < kPairListPer; ++z)
      if (v[z] != kNotFirst) l.touched[at++] = v[z] < 0 ? ~v[z] : v[z];
    total += all;
  }
  const int is = tid < kWindows ? s_long[min(tid, kWindows - 1)] : 0;
  int4 m{};
  if (is) m = l.multi[tid];
  int n_multi;
  const int at = block_excl_scan_256(is, s_w, n_multi);   // (every entry has been read before one is written)
  if (is) l.multi[at] = m;
  if (tid == 0) { *l.n_touched = total; l.totals[0] = total; l.totals[2] = n_multi; }
}

// Work of the two kernels below: units of (run of consecutive chunks, 1 KB of columns).  The pairs of a run are consecutive in
// the grouped list, whatever their neurons, so a wave reads the list 64 pairs and the rows eight pairs at a time and starts a
// new sum where a chunk ends; a wave per chunk (eight pairs on average where each of 2048 tokens selects 256 of 65536
// neurons, one or two elsewhere) spent more on finding its pairs and waiting for them than on the rows: both
// kernels 1070 us there, as runs 770.
// The units are dealt to the XCDs by columns: XCD x takes the x-th eighth of them, ordered by columns first.  Where 2048 bf16
// tokens have 4096 columns, that is one slice of 2 MB of h or dOut per XCD, which stays in its L2, so that the row reads, one per
// (token, neuron) pair, do not go to memory.  The waves of an XCD take its units in turn (workgroup ids go to the XCDs in turn;
// gridDim.x is a multiple of 8).
// Where pair_one_kernel left the entries (kGaps), a run is that of consecutive entries, of which some hold no chunk.
constexpr int kSegWorkgroups = 5 * 256;   // what the registers of either kernel let the compute units hold
constexpr int kSegRun = 16;               // entries per run at most; fewer where that leaves waves without one

struct SegRuns {
  long long unit, end;
  int slice, run, n_runs, len, step;
  // Workgroup wg of n_wg; n_wg and the number of the launch's first a multiple of 8.  `entries` work entries per chunk.
  __device__ __forceinline__ bool init(int n_entries, int entries, int n_slices, int wg, int n_wg) {
    const long long share = (long long)(n_entries / entries) * n_slices / (kSegWorkgroups * 4);
    len = min((share < 1 ? 1 : share > kSegRun ? kSegRun : (int)share) * entries, 64);
    n_runs = (n_entries + len - 1) / len;
    const long long units = (long long)n_runs * n_slices, per = (units + 7) / 8;
    const int x = wg & 7;
    step = (n_wg >> 3) * 4;
    unit = x * per + (wg >> 3) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    end = min((x + 1) * per, units);
    if (unit >= end) return false;
    slice = (int)(unit / n_runs);
    run = (int)(unit - (long long)slice * n_runs);
    return true;
  }
  __device__ __forceinline__ bool next() {
    unit += step;
    run += step;
    while (run >= n_runs) { run -= n_runs; ++slice; }
    return unit < end;
  }
};

// The chunks of entries c0 .. c0 + m - 1 (m <= 64): lane i receives the i-th; returns their number, which may be 0 where there are gaps.
template <bool kGaps>
__device__ __forceinline__ int seg_run_chunks(const SegWork* __restrict__ work, int c0, int m, SegWork& w) {
  const int lane = threadIdx.x & 63;
  w = work[c0 + min(lane, m - 1)];
  if constexpr (!kGaps) return m;
  const bool is = lane < m && w.len > 0;
  const unsigned long long mask = __ballot(is), before = (1ull << lane) - 1ull;
  const int n = __popcll(mask), to = 4 * (is ? __popcll(mask & before) : n + __popcll(~mask & before));
  w.j = __builtin_amdgcn_ds_permute(to, w.j);
  w.off = __builtin_amdgcn_ds_permute(to, w.off);
  w.len = __builtin_amdgcn_ds_permute(to, w.len);
  w.part = __builtin_amdgcn_ds_permute(to, w.part);
  return n;
}

// Up to this many partial dot products per pair (one per group of column slices)
constexpr int kDsParts = 8;

// dV of a run of chunks over one slice of columns, and with the same dOut rows the slice's part of ds = dOut[t,:] . V[j,:],
// left in ds_part[group of slices][position of the pair in the list].  A neuron of one chunk gets its row written here; the
// chunks of a longer segment leave their fp32 sums in `part` ([chunk][dV | dK][d]), which are added in chunk order later.
// What bounds it: vector arithmetic (about 30 instructions per pair and KB of row), V read and dV written, and the rows out of
// L2 about alike.  The activation gradients used to be formed token by token, which reads a row of V per pair from beyond L2; with
// that gone: 2048 tokens x 256 pairs, d 4096, bf16, 65536 neurons: backward 1780 -> 1340 us (this kernel 460, dK 310, dh 550); 2048 x
// 64 pairs, d 768, fp32, 8192 neurons: 180 -> 113.
template <typename T, bool kGaps>
__global__ __launch_bounds__(256, 5) void seg_dv_kernel(const SegWork* __restrict__ work, const int32_t* __restrict__ totals,
                                                        const int2* __restrict__ seg, const T* __restrict__ V,
                                                        const T* __restrict__ dOut, int d, int n_slices, size_t n_pairs,
                                                        T* __restrict__ dV, float* __restrict__ part,
                                                        float* __restrict__ ds_part, int entries, PairLists lists) {
  constexpr int VE = Vec16<T>::kElems;
  int wg = blockIdx.x, n_wg = gridDim.x;
  if constexpr (kGaps) {   // the first eight workgroups: the lists
    if (wg == 0) pair_lists_body(lists);
    if (wg < 8) return;
    wg -= 8; n_wg -= 8;
  }
  const int lane = threadIdx.x & 63, n_groups = n_slices < kDsParts ? n_slices : kDsParts;
  const int n_chunks = kGaps ? (int)n_pairs : totals[1];
  SegRuns cur;   // (its slices are the groups of slices)
  for (bool more = cur.init(n_chunks, entries, n_groups, wg, n_wg); more; more = cur.next()) {
    const int c0 = cur.run * cur.len;
    SegWork w;   // lane: its chunk of the run
    const int nc = seg_run_chunks<kGaps>(work, c0, min(cur.len, n_chunks - c0), w);
    if (kGaps && nc == 0) continue;
    const int beg = __builtin_amdgcn_readlane(w.off, 0);
    const int end = __builtin_amdgcn_readlane(w.off, nc - 1) + __builtin_amdgcn_readlane(w.len, nc - 1);
    float* dsp = ds_part + cur.slice * n_pairs;
    for (int slice = cur.slice; slice < n_slices; slice += n_groups) {
      const int col = (slice * 64 + lane) * VE, at = min(col, d - VE);
      auto v_row = [&](int c) {
        return *reinterpret_cast<const u32x4*>(V + (size_t)__builtin_amdgcn_readlane(w.j, min(c, nc - 1)) * d + at);
      };
      int ci = 0, stop = beg + __builtin_amdgcn_readlane(w.len, 0);   // the chunk that is worked on, and where it ends
      float v[VE], aV[VE];
      Vec16<T>::unpack(v_row(0), v);
      u32x4 v_next = v_row(1);   // (asking for the V rows of all chunks that begin in a batch with its rows gained nothing)
#pragma unroll
      for (int c = 0; c < VE; ++c) aV[c] = 0.f;
      auto flush = [&]() {
        const int row = __builtin_amdgcn_readlane(w.j, ci), to = __builtin_amdgcn_readlane(w.part, ci);
        if (col < d) {
          if (to < 0) Vec16<T>::store(dV + (size_t)row * d + col, aV);
          else Vec16<T>::store_f32(part + (size_t)to * 2 * d + col, aV);
        }
      };
      for (int i0 = beg; i0 < end; i0 += 64) {
        const int n = min(64, end - i0);
        const int2 e = seg[i0 + min(lane, n - 1)];
        for (int q = 0; q < n; q += 8) {
          u32x4 g[8];
          float dot[8];
#pragma unroll
          for (int u = 0; u < 8; ++u)
            g[u] = *reinterpret_cast<const u32x4*>(dOut + (size_t)__builtin_amdgcn_readlane(e.x, min(q + u, n - 1)) * d + at);
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            dot[u] = 0.f;
            if (q + u < n) {
              if (i0 + q + u == stop) {   // the next chunk's first pair
                flush();
                ++ci;
                stop += __builtin_amdgcn_readlane(w.len, ci);
                Vec16<T>::unpack(v_next, v);
                v_next = v_row(ci + 1);
#pragma unroll
                for (int c = 0; c < VE; ++c) aV[c] = 0.f;
              }
              const float a = __int_as_float(__builtin_amdgcn_readlane(e.y, q + u));
              float y[VE];
              Vec16<T>::unpack(g[u], y);
#pragma unroll
              for (int c = 0; c < VE; ++c) {
                aV[c] = fmaf(a, y[c], aV[c]);
                dot[u] = fmaf(y[c], v[c], dot[u]);
              }
              dot[u] = col < d ? dot[u] : 0.f;
            }
          }
          const float r = wave_sum8(dot);
          if (lane < 8 && q + lane < n) {
            float* o = dsp + i0 + q + lane;
            *o = slice == cur.slice ? r : *o + r;
          }
        }
      }
      flush();
    }
  }
}

// ds of the pairs from their parts, in slice order, and dK of a run of chunks over one slice of columns.  ds == nullptr: not
// wanted in token order.
template <typename T, bool kGaps>
__global__ __launch_bounds__(256, 6) void seg_dk_kernel(const SegWork* __restrict__ work, const int32_t* __restrict__ totals,
                                                        const int2* __restrict__ seg, const int32_t* __restrict__ pair_sorted,
                                                        const float* __restrict__ ds_part, const T* __restrict__ h, int d,
                                                        int n_slices, size_t n_pairs, T* __restrict__ dK,
                                                        float* __restrict__ part, float* __restrict__ ds, int entries) {
  constexpr int VE = Vec16<T>::kElems;
  const int lane = threadIdx.x & 63, n_parts = n_slices < kDsParts ? n_slices : kDsParts;
  const int n_chunks = kGaps ? (int)n_pairs : totals[1];
  SegRuns cur;
  for (bool more = cur.init(n_chunks, entries, n_slices, blockIdx.x, gridDim.x); more; more = cur.next()) {
    const int c0 = cur.run * cur.len;
    SegWork w;
    const int nc = seg_run_chunks<kGaps>(work, c0, min(cur.len, n_chunks - c0), w);
    if (kGaps && nc == 0) continue;
    const int beg = __builtin_amdgcn_readlane(w.off, 0);
    const int end = __builtin_amdgcn_readlane(w.off, nc - 1) + __builtin_amdgcn_readlane(w.len, nc - 1);
    const int col = (cur.slice * 64 + lane) * VE, at = min(col, d - VE);
    int ci = 0, stop = beg + __builtin_amdgcn_readlane(w.len, 0);
    float aK[VE];
#pragma unroll
    for (int c = 0; c < VE; ++c) aK[c] = 0.f;
    auto flush = [&]() {
      const int row = __builtin_amdgcn_readlane(w.j, ci), to = __builtin_amdgcn_readlane(w.part, ci);
      if (col < d) {
        if (to < 0) Vec16<T>::store(dK + (size_t)row * d + col, aK);
        else Vec16<T>::store_f32(part + (size_t)to * 2 * d + d + col, aK);
      }
    };
    for (int i0 = beg; i0 < end; i0 += 64) {
      const int n = min(64, end - i0), i = i0 + min(lane, n - 1);
      const int2 e = seg[i];
      float p[kDsParts];
#pragma unroll
      for (int g = 0; g < kDsParts; ++g) p[g] = g < n_parts ? ds_part[g * n_pairs + i] : 0.f;
      float s = p[0];
#pragma unroll
      for (int g = 1; g < kDsParts; ++g) s += p[g];
      s = __int_as_float(e.y) > 0.f ? s : 0.f;
      if (cur.slice == 0 && ds != nullptr && lane < n) ds[pair_sorted[i]] = s;
      for (int q = 0; q < n; q += 8) {
        u32x4 rows[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
          rows[u] = *reinterpret_cast<const u32x4*>(h + (size_t)__builtin_amdgcn_readlane(e.x, min(q + u, n - 1)) * d + at);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          if (q + u < n) {
            if (i0 + q + u == stop) {
              flush();
              ++ci;
              stop += __builtin_amdgcn_readlane(w.len, ci);
#pragma unroll
              for (int c = 0; c < VE; ++c) aK[c] = 0.f;
            }
            const float cf = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(s), q + u));
            float y[VE];
            Vec16<T>::unpack(rows[u], y);
#pragma unroll
            for (int c = 0; c < VE; ++c) aK[c] = fmaf(cf, y[c], aK[c]);
          }
        }
      }
    }
    flush();
  }
}

// dV, ds and dK of a chunk at once, where there is little to do: 2^lg waves of a workgroup take the chunk, each every 2^lg-th KB of
// its columns; a part of ds per wave goes through LDS, the parts are added in wave order.  Up to kSegAhead rows of h are asked for with
// those of dOut.  Work entries may be empty (pair_one_kernel); a wave looks at 64 of the workgroup's at a time.
// Bound by the chain of loads per chunk (entry, pairs, rows), which a launch less outweighs only while waves have few chunks each:
// see seg_rows_fused.
constexpr int kSegAhead = 4;
constexpr int kSegRowsWgs = 4 * 256;   // what the registers let the compute units hold
template <typename T>
__global__ __launch_bounds__(256, 4) void seg_rows_kernel(const SegWork* __restrict__ work, const int32_t* __restrict__ totals,
                                                          int n_pairs, const int2* __restrict__ seg,
                                                          const int32_t* __restrict__ pair_sorted, const T* __restrict__ V,
                                                          const T* __restrict__ dOut, const T* __restrict__ h, int d, int n_slices,
                                                          int lg, T* __restrict__ dV, T* __restrict__ dK,
                                                          float* __restrict__ part, float* __restrict__ ds, PairLists lists) {
  constexpr int VE = Vec16<T>::kElems;
  __shared__ float s_ds[2][4][kSegChunk];
  int wg = blockIdx.x, n_wg = gridDim.x;
  if (lists.first != nullptr) {
    if (wg == 0) {
      pair_lists_body(lists);
      return;
    }
    --wg; --n_wg;
  }
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int G = 1 << lg, g = wave & (G - 1), group = wave >> lg, w0 = wave - g;
  const int n = lists.first != nullptr ? n_pairs : totals[1], per = (n + n_wg - 1) / n_wg;
  const int end = min(n, (wg + 1) * per);
  int buf = 0;
  for (int c0 = wg * per; c0 < end; c0 += 64) {
    const int m = min(64, end - c0);
    const SegWork e = work[c0 + min(lane, m - 1)];
    unsigned long long live = __ballot(lane < m && e.len > 0);   // the same in every wave
    while (live) {
      int c = -1;   // this wave's entry: the group-th of the next ones
      for (int z = 0; z < 4 >> lg; ++z) {
        if (z == group && live) c = __ffsll(live) - 1;
        live &= live - 1;
      }
      const bool has = c >= 0;
      const int cc = max(c, 0);
      const int j = __builtin_amdgcn_readlane(e.j, cc), off = __builtin_amdgcn_readlane(e.off, cc),
                len = has ? __builtin_amdgcn_readlane(e.len, cc) : 0, to = __builtin_amdgcn_readlane(e.part, cc);
      u32x4 hx[kSegAhead];
      auto sum_v = [&](auto batch) {
        constexpr int U = decltype(batch)::value;
        for (int slice = g; slice < n_slices; slice += G) {
          const int col = (slice * 64 + lane) * VE, at = min(col, d - VE);
          float v[VE], aV[VE];
          const u32x4 v_row = *reinterpret_cast<const u32x4*>(V + (size_t)j * d + at);
#pragma unroll
          for (int x = 0; x < VE; ++x) aV[x] = 0.f;
          for (int i0 = 0; i0 < len; i0 += 64) {
            const int np = min(64, len - i0);
            const int2 p = seg[off + i0 + min(lane, np - 1)];
            for (int q = 0; q < np; q += U) {
              u32x4 rows[U];
              float dot[8];
#pragma unroll
              for (int u = 0; u < U; ++u)
                rows[u] = *reinterpret_cast<const u32x4*>(dOut + (size_t)__builtin_amdgcn_readlane(p.x, min(q + u, np - 1)) * d + at);
              if constexpr (U <= kSegAhead) {
                if (slice == g) {
#pragma unroll
                  for (int u = 0; u < U; ++u)
                    hx[u] = *reinterpret_cast<const u32x4*>(h + (size_t)__builtin_amdgcn_readlane(p.x, min(u, np - 1)) * d + at);
                }
              }
              Vec16<T>::unpack(v_row, v);
#pragma unroll
              for (int u = 0; u < 8; ++u) {
                dot[u] = 0.f;
                if (u < U && q + u < np) {
                  const float a = __int_as_float(__builtin_amdgcn_readlane(p.y, q + u));
                  float y[VE];
                  Vec16<T>::unpack(rows[u % U], y);
#pragma unroll
                  for (int x = 0; x < VE; ++x) {
                    aV[x] = fmaf(a, y[x], aV[x]);
                    dot[u] = fmaf(y[x], v[x], dot[u]);
                  }
                  dot[u] = col < d ? dot[u] : 0.f;
                }
              }
              const float r = wave_sum8(dot);
              if (lane < U && q + lane < np) {
                float* o = &s_ds[buf][wave][i0 + q + lane];
                *o = slice == g ? r : *o + r;
              }
            }
          }
          if (col < d) {
            if (to < 0) Vec16<T>::store(dV + (size_t)j * d + col, aV);
            else Vec16<T>::store_f32(part + (size_t)to * 2 * d + col, aV);
          }
        }
      };
      auto sum_k = [&](auto batch) {
        constexpr int U = decltype(batch)::value;
        for (int slice = g; slice < n_slices; slice += G) {
          const int col = (slice * 64 + lane) * VE, at = min(col, d - VE);
          float aK[VE];
#pragma unroll
          for (int x = 0; x < VE; ++x) aK[x] = 0.f;
          for (int i0 = 0; i0 < len; i0 += 64) {
            const int np = min(64, len - i0), i = i0 + min(lane, np - 1);
            const int2 p = seg[off + i];
            float s = s_ds[buf][w0][i];
            for (int z = 1; z < min(G, n_slices); ++z) s += s_ds[buf][w0 + z][i];
            s = __int_as_float(p.y) > 0.f ? s : 0.f;
            if (slice == 0 && ds != nullptr && lane < np) ds[pair_sorted[off + i]] = s;
            for (int q = 0; q < np; q += U) {
              u32x4 rows[U];
              if (U > kSegAhead || slice != g) {
#pragma unroll
                for (int u = 0; u < U; ++u)
                  rows[u] = *reinterpret_cast<const u32x4*>(h + (size_t)__builtin_amdgcn_readlane(p.x, min(q + u, np - 1)) * d + at);
              } else if constexpr (U <= kSegAhead) {
#pragma unroll
                for (int u = 0; u < U; ++u) rows[u] = hx[u];
              }
#pragma unroll
              for (int u = 0; u < U; ++u) {
                if (q + u < np) {
                  const float cf = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(s), q + u));
                  float y[VE];
                  Vec16<T>::unpack(rows[u], y);
#pragma unroll
                  for (int x = 0; x < VE; ++x) aK[x] = fmaf(cf, y[x], aK[x]);
                }
              }
            }
          }
          if (col < d) {
            if (to < 0) Vec16<T>::store(dK + (size_t)j * d + col, aK);
            else Vec16<T>::store_f32(part + (size_t)to * 2 * d + d + col, aK);
          }
        }
      };
      // (rows asked for twice cost as much as others: batches of what there is)
      if (len == 1) sum_v(std::integral_constant<int, 1>{});
      else if (len == 2) sum_v(std::integral_constant<int, 2>{});
      else if (len > 0 && len <= kSegAhead) sum_v(std::integral_constant<int, kSegAhead>{});
      else if (len > 0) sum_v(std::integral_constant<int, 8>{});
      if (G > 1) __syncthreads();
      else wave_lds_fence();
      if (len == 1) sum_k(std::integral_constant<int, 1>{});
      else if (len == 2) sum_k(std::integral_constant<int, 2>{});
      else if (len > 0 && len <= kSegAhead) sum_k(std::integral_constant<int, kSegAhead>{});
      else if (len > 0) sum_k(std::integral_constant<int, 8>{});
      buf ^= 1;   // (one barrier per entry: the other half is written before this one has been read by all)
    }
  }
}

// The rows of the touched neurons of more than one chunk: their chunks' partial sums added in chunk order.  Executed by
// workgroup `wg` of n_wg.
template <typename T>
__device__ __forceinline__ void seg_finish_body(int wg, int n_wg, const int4* __restrict__ multi, const int32_t* __restrict__ totals,
                                                const float* __restrict__ part, int d, T* __restrict__ dK, T* __restrict__ dV) {
  for (int u = wg; u < totals[2]; u += n_wg) {
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
