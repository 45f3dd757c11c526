// Backward of the per-pair path without floating-point atomics: the (token, neuron) pairs are grouped by neuron (counting
// sort; integer atomics only decide positions, and every group is then put in ascending pair order, i.e. ascending token),
// and the group is worked through in that fixed order, in chunks of kSegChunk pairs (a wave per chunk and 1 KB of columns;
// the chunk sums of a long group are added in chunk order):
//   dV[j,:] = sum act * dOut[t,:],  ds = act > 0 ? dOut[t,:] . V[j,:] : 0,  dK[j,:] = sum ds * h[t,:].
// Only touched rows are written.  A token's dh, the sum of ds * K[j,:] over its pairs, follows in gather.h.
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
// neurons of more than one chunk}.  A workgroup of 1024 threads takes kScanChunk counters and adds up the ones before them
// itself, out of L2 (65536 neurons: 119 us by one workgroup for all of them, 16 us with 256 threads, 15 us with 1024), or, beyond
// kScanSelfMax counters, takes the sums that pair_sums_kernel left.
constexpr int kScanChunk = 2048, kScanSelfMax = 1 << 17, kScanThreads = 1024, kScanPer = kScanChunk / kScanThreads;
struct PairSums {
  int c, f, wk, mu, mn;   // pairs, touched neurons, chunks, chunks of neurons with several, such neurons
  __device__ __forceinline__ void add(int v) {
    const int ch = (v + kSegChunk - 1) / kSegChunk;
    c += v; f += v > 0; wk += ch; mu += ch > 1 ? ch : 0; mn += ch > 1 ? 1 : 0;
  }
};

// sums over a workgroup of kScanThreads threads, in every thread
__device__ __forceinline__ PairSums pair_sums_all(PairSums x, int (*s)[kScanThreads / 64]) {
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
  for (int z = 0; z < 5; ++z) {
    r[z] = 0;
#pragma unroll
    for (int i = 0; i < kScanThreads / 64; ++i) r[z] += s[z][i];
  }
  __syncthreads();
  return PairSums{r[0], r[1], r[2], r[3], r[4]};
}

__global__ __launch_bounds__(kScanThreads) void pair_sums_kernel(const int32_t* __restrict__ cnt, int N, PairSums* __restrict__ sums) {
  __shared__ int s[5][kScanThreads / 64];
  PairSums x{0, 0, 0, 0, 0};
  const int j0 = blockIdx.x * kScanChunk + threadIdx.x * kScanPer;
#pragma unroll
  for (int z = 0; z < kScanPer; ++z)
    if (j0 + z < N) x.add(cnt[j0 + z]);
  x = pair_sums_all(x, s);
  if (threadIdx.x == 0) sums[blockIdx.x] = x;
}

__global__ __launch_bounds__(kScanThreads) void pair_scan_kernel(const int32_t* __restrict__ cnt, int N,
                                                        const PairSums* __restrict__ sums,
                                                        int32_t* __restrict__ seg_off, int32_t* __restrict__ touched,
                                                        int32_t* __restrict__ n_touched, SegWork* __restrict__ work,
                                                        int4* __restrict__ multi, int32_t* __restrict__ totals) {
  __shared__ int s[5][kScanThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, chunk = blockIdx.x;
  PairSums before{0, 0, 0, 0, 0};
  if (sums != nullptr) {
    for (int c = tid; c < chunk; c += kScanThreads) {
      const PairSums y = sums[c];
      before.c += y.c; before.f += y.f; before.wk += y.wk; before.mu += y.mu; before.mn += y.mn;
    }
  } else {
    const i32x4* c4 = reinterpret_cast<const i32x4*>(cnt);
#pragma unroll 4
    for (int c = tid; c < chunk * (kScanChunk / 4); c += kScanThreads) {
      const i32x4 v = c4[c];
      before.add(v.x); before.add(v.y); before.add(v.z); before.add(v.w);
    }
  }
  before = pair_sums_all(before, s);
  const int j0 = chunk * kScanChunk + tid * kScanPer;
  int v[kScanPer];
  PairSums mine{0, 0, 0, 0, 0};
#pragma unroll
  for (int z = 0; z < kScanPer; ++z) {
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

// All of the above in one launch: up to kPairOneP pairs of kPairOneN neurons.  Every workgroup counts all pairs in LDS, eight a
// thread, and scans all counters; neuron j belongs to workgroup j % kPairOneWgs, which writes its work entries and puts its pairs
// in order.  The five launches that this replaces depend on each other and take 4-7 us each, however few the pairs.
// fp32 steps, five launches / one: 78 tokens x 4 pairs, 2496 neurons 53.5 -> 41 us; 124 x 37, 7872 neurons 56.5 -> 51.  More pairs
// than a thread's eight would have to be read again for every step: in that form 9937 pairs gained 2 us and 64000 lost 11 of 140.
constexpr int kPairOnePairs = 8, kPairOneP = kPairOnePairs * kScanThreads, kPairOneN = 1 << 14, kPairOneWgs = 128;
constexpr int kPairOnePer = kPairOneN / kScanThreads;   // consecutive counters of a thread
constexpr int kPairOneLds = kPairOneN + kPairOneN / kPairOnePer + 1;
__global__ __launch_bounds__(kScanThreads) void pair_one_kernel(const int32_t* __restrict__ idx, const float* __restrict__ act, int P,
                                                       int N, int k, int32_t* __restrict__ touched,
                                                       int32_t* __restrict__ n_touched, SegWork* __restrict__ work,
                                                       int4* __restrict__ multi, int32_t* __restrict__ totals,
                                                       int32_t* __restrict__ pair_sorted, int2* __restrict__ seg) {
  constexpr int kPer = kPairOnePer, kThreads = kScanThreads;
  static_assert(kPer <= kPairOneWgs && kPairOneP <= kBitonicMax && (long long)kPairOneP * kPairOneN <= 1ll << 31, "");   // at most one of a thread's counters is the workgroup's
  extern __shared__ int32_t s_cnt[];   // counts, then first places; neuron j at j + j / kPer, so that the scan's reads spread over the banks
  __shared__ __attribute__((aligned(16))) int32_t s_p[kBitonicMax];
  __shared__ int32_t s_list[kPairOneP];   // this workgroup's segments, where they are in the grouped list
  __shared__ int32_t s_long[kPairOneN / kPairOneWgs], s_sum[5][kThreads / 64], s_n, s_nlong;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, wg = blockIdx.x;
  auto slot = [](int j) { return j + j / kPer; };
  auto mine = [&](int j) { return j % kPairOneWgs == wg; };
  int jp[kPairOnePairs], at[kPairOnePairs];   // of the pairs tid + kThreads * z: neuron, place among the neuron's as they come
#pragma unroll
  for (int z = 0; z < kPairOnePairs; ++z) jp[z] = idx[min(tid + kThreads * z, P - 1)];
  for (int i = tid; i <= slot(N); i += kThreads) s_cnt[i] = 0;
  if (tid == 0) s_n = s_nlong = 0;
  __syncthreads();
#pragma unroll
  for (int z = 0; z < kPairOnePairs; ++z) {
    jp[z] = tid + kThreads * z < P ? clampi(jp[z], 0, N - 1) : -1;
    at[z] = jp[z] >= 0 ? atomicAdd(&s_cnt[slot(jp[z])], 1) : 0;
  }
  __syncthreads();
  const int j0 = tid * kPer;
  int v[kPer];
  PairSums sum{0, 0, 0, 0, 0};
#pragma unroll
  for (int z = 0; z < kPer; ++z) {
    v[z] = j0 + z < N ? s_cnt[slot(j0 + z)] : 0;
    sum.add(v[z]);
  }
  const int m[5] = {sum.c, sum.f, sum.wk, sum.mu, sum.mn};
  int ex[5];
#pragma unroll
  for (int z = 0; z < 5; ++z) {
    const int incl = wave_incl_scan(m[z]);
    if (lane == 63) s_sum[z][w] = incl;
    ex[z] = incl - m[z];
  }
  __syncthreads();
#pragma unroll
  for (int z = 0; z < 5; ++z)
    for (int i = 0; i < w; ++i) ex[z] += s_sum[z][i];
  int off = ex[0], nt = ex[1], wo = ex[2], mo = ex[3], mn = ex[4];
#pragma unroll
  for (int z = 0; z < kPer; ++z) {
    const int j = j0 + z, ch = (v[z] + kSegChunk - 1) / kSegChunk;
    if (j < N) s_cnt[slot(j)] = off;
    if (v[z] > 0 && mine(j)) {
      touched[nt] = j;
      if (ch > 1) multi[mn] = make_int4(j, mo, ch, 0);
      for (int c = 0; c < ch; ++c)
        work[wo + c] = SegWork{j, off + c * kSegChunk, min(v[z] - c * kSegChunk, kSegChunk), ch > 1 ? mo + c : -1};
      if (ch > 1) s_long[atomicAdd(&s_nlong, 1)] = j;
    }
    off += v[z]; nt += v[z] > 0 ? 1 : 0; wo += ch; mo += ch > 1 ? ch : 0; mn += ch > 1 ? 1 : 0;
  }
  if (tid == kThreads - 1) {
    s_cnt[slot(N)] = off;   // (behind every counter)
    if (wg == 0) { *n_touched = nt; totals[0] = nt; totals[1] = wo; totals[2] = mn; }
  }
  __syncthreads();
#pragma unroll
  for (int z = 0; z < kPairOnePairs; ++z)
    if (jp[z] >= 0 && mine(jp[z])) {
      s_list[s_cnt[slot(jp[z])] + at[z]] = tid + kThreads * z;
      s_p[atomicAdd(&s_n, 1)] = (tid + kThreads * z) * kPairOneN + jp[z];
    }
  __syncthreads();
  auto put = [&](int i, int p) {
    pair_sorted[i] = p;
    seg[i] = make_int2(p / k, __float_as_int(act[p]));
  };
  // (a thread per pair of the workgroup: left where they are, a wave would rank its few one after the other)
  for (int i = tid; i < s_n; i += kThreads) {
    const int p = s_p[i] / kPairOneN, j = s_p[i] % kPairOneN, o = s_cnt[slot(j)], L = s_cnt[slot(j + 1)] - o;
    if (L > kSegChunk) continue;
    int r = 0;
#pragma unroll 4
    for (int y = 0; y < L; ++y) r += s_list[o + y] < p ? 1 : 0;
    put(o + r, p);
  }
  __syncthreads();
  for (int u = 0; u < s_nlong; ++u) {
    const int j = s_long[u], o = s_cnt[slot(j)];
    sort_long_segment<kThreads>(s_list + o, s_cnt[slot(j + 1)] - o, s_p, [&](int i, int p) { put(o + i, p); });
  }
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
constexpr int kSegWorkgroups = 5 * 256;   // what the registers of either kernel let the compute units hold
constexpr int kSegRun = 16;               // chunks per run at most; fewer where that leaves waves without one

struct SegRuns {
  long long unit, end;
  int slice, run, n_runs, len, step;
  __device__ __forceinline__ bool init(int n_chunks, int n_slices) {
    const long long share = (long long)n_chunks * n_slices / (kSegWorkgroups * 4);
    len = share < 1 ? 1 : share > kSegRun ? kSegRun : (int)share;
    n_runs = (n_chunks + len - 1) / len;
    const long long units = (long long)n_runs * n_slices, per = (units + 7) / 8;
    const int x = blockIdx.x & 7;
    step = (int)(gridDim.x >> 3) * 4;
    unit = x * per + (int)(blockIdx.x >> 3) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
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

// Up to this many partial dot products per pair (one per group of column slices)
constexpr int kDsParts = 8;

// dV of a run of chunks over one slice of columns, and with the same dOut rows the slice's part of ds = dOut[t,:] . V[j,:],
// left in ds_part[group of slices][position of the pair in the list].  A neuron of one chunk gets its row written here; the
// chunks of a longer segment leave their fp32 sums in `part` ([chunk][dV | dK][d]), which are added in chunk order later.
// What bounds it: vector arithmetic (about 30 instructions per pair and KB of row), V read and dV written, and the rows out of
// L2 about alike.  The activation gradients used to be formed token by token, which reads a row of V per pair from beyond L2; with
// that gone: 2048 tokens x 256 pairs, d 4096, bf16, 65536 neurons: backward 1780 -> 1340 us (this kernel 460, dK 310, dh 550); 2048 x
// 64 pairs, d 768, fp32, 8192 neurons: 180 -> 113.
template <typename T>
__global__ __launch_bounds__(256, 5) void seg_dv_kernel(const SegWork* __restrict__ work, const int32_t* __restrict__ totals,
                                                        const int2* __restrict__ seg, const T* __restrict__ V,
                                                        const T* __restrict__ dOut, int d, int n_slices, size_t n_pairs,
                                                        T* __restrict__ dV, float* __restrict__ part,
                                                        float* __restrict__ ds_part) {
  constexpr int VE = Vec16<T>::kElems;
  const int lane = threadIdx.x & 63, n_groups = n_slices < kDsParts ? n_slices : kDsParts;
  const int n_chunks = totals[1];
  SegRuns cur;   // (its slices are the groups of slices)
  for (bool more = cur.init(n_chunks, n_groups); more; more = cur.next()) {
    const int c0 = cur.run * cur.len, nc = min(cur.len, n_chunks - c0);
    const SegWork w = work[c0 + min(lane, nc - 1)];   // lane: its chunk of the run
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
template <typename T>
__global__ __launch_bounds__(256, 6) void seg_dk_kernel(const SegWork* __restrict__ work, const int32_t* __restrict__ totals,
                                                        const int2* __restrict__ seg, const int32_t* __restrict__ pair_sorted,
                                                        const float* __restrict__ ds_part, const T* __restrict__ h, int d,
                                                        int n_slices, size_t n_pairs, T* __restrict__ dK,
                                                        float* __restrict__ part, float* __restrict__ ds) {
  constexpr int VE = Vec16<T>::kElems;
  const int lane = threadIdx.x & 63, n_parts = n_slices < kDsParts ? n_slices : kDsParts;
  const int n_chunks = totals[1];
  SegRuns cur;
  for (bool more = cur.init(n_chunks, n_slices); more; more = cur.next()) {
    const int c0 = cur.run * cur.len, nc = min(cur.len, n_chunks - c0);
    const SegWork w = work[c0 + min(lane, nc - 1)];
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
