// The per-pair path's sums over a token's pairs: the value sum of the forward (Eq. 4), out[t,:] = sum_i act[t,i] V[idx[t,i],:],
// and in the backward dh[t,:] = sum_i ds[t,i] K[idx[t,i],:].
#pragma once
#include "common.h"
#include "scatter.h"

namespace meft {

// What the launch does besides (backward): the rows of neurons of more than one chunk, by the first n_wg workgroups.
template <typename T>
struct SegFinish {
  int n_wg;   // a multiple of 8, or 0
  const int4* multi;
  const int32_t* totals;
  const float* part;
  T *dK, *dV;
};

// row[t,:] = sum over the token's pairs of coef * W[idx,:], fp32: kAcc sums, of the pairs kAcc apart in list order, which are
// added at the end.  gate: pairs whose gate is not positive are left out (their W row is not read); nullptr: none.
// U: rows a wave asks for together: 8, or as few as a token has pairs (a row asked for twice costs as much as another: 10000
// tokens x 1 pair, d 4096, fp32, backward 249 -> 216 us).
// A wave takes (token, 1 KB of columns), a workgroup four tokens of the same columns, and the columns are dealt to the XCDs: XCD
// x takes the x-th eighth of the units, ordered by columns first.  The tokens' lists ascend (the selection writes them so), and
// the waves of an XCD go through them side by side, so a row's KB that several tokens selected is asked for by them within a short
// time; they drift further apart than an L2 holds all the same: of 4.3 GB of rows an eighth is found there (3.7 GB come from beyond
// it, at 7 TB/s).  A compute unit has about a hundred 128-byte lines in flight, so what counts is how soon a line is there.  2048
// tokens x 256 pairs, d 4096, bf16, 65536 neurons: 575 -> 510 us; 1000 x 64, d 768, fp32, 8192 neurons: 22 -> 16.
template <typename T, int kAcc, int U>
__global__ __launch_bounds__(256) void pair_rows_kernel(const T* __restrict__ W, const int32_t* __restrict__ idx,
                                                        const float* __restrict__ coef, const float* __restrict__ gate,
                                                        int n_tok, int d, int k, int N, T* __restrict__ row, SegFinish<T> f) {
  constexpr int VE = Vec16<T>::kElems;
  long long w = (long long)blockIdx.y * gridDim.x + blockIdx.x;
  if (w < f.n_wg) {
    seg_finish_body<T>((int)w, f.n_wg, f.multi, f.totals, f.part, d, f.dK, f.dV);
    return;
  }
  w -= f.n_wg;
  const int groups = (n_tok + 3) / 4, n_slices = (d + 64 * VE - 1) / (64 * VE);
  const long long units = (long long)groups * n_slices, per = (units + 7) / 8, unit = (w & 7) * per + (w >> 3);
  if ((w >> 3) >= per || unit >= units) return;
  const int slice = (int)(unit / groups);
  const int t = (int)(unit - (long long)slice * groups) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (t >= n_tok) return;
  const int lane = threadIdx.x & 63;
  const int col = slice * 64 * VE + lane * VE, at = min(col, d - VE);
  float acc[kAcc][VE];
#pragma unroll
  for (int a = 0; a < kAcc; ++a)
#pragma unroll
    for (int c = 0; c < VE; ++c) acc[a][c] = 0.f;
  for (int i0 = 0; i0 < k; i0 += 64) {
    const int n = min(64, k - i0);
    const size_t p = (size_t)t * k + i0 + min(lane, n - 1);
    const int j = clampi(idx[p], 0, N - 1);
    const float cf = coef[p];
    unsigned long long live = __ballot(lane < n && (gate == nullptr || gate[p] > 0.f));
    while (live) {
      u32x4 x[U];
      int at_u[U];
      const int m = min(U, (int)__popcll(live));
#pragma unroll
      for (int u = 0; u < U; ++u) {
        at_u[u] = live ? __ffsll(live) - 1 : at_u[u > 0 ? u - 1 : 0];
        live &= live - 1;
        x[u] = *reinterpret_cast<const u32x4*>(W + (size_t)__builtin_amdgcn_readlane(j, at_u[u]) * d + at);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (u < m) {
          const float c1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cf), at_u[u]));
          float y[VE];
          Vec16<T>::unpack(x[u], y);
#pragma unroll
          for (int c = 0; c < VE; ++c) acc[u % kAcc][c] = fmaf(c1, y[c], acc[u % kAcc][c]);
        }
      }
    }
  }
#pragma unroll
  for (int a = 1; a < kAcc; ++a)
#pragma unroll
    for (int c = 0; c < VE; ++c) acc[0][c] += acc[a][c];
  if (col < d) Vec16<T>::store(row + (size_t)t * d + col, acc[0]);
}

}  // namespace meft
