// Small token groups on the block-dense path.  The router does not balance its blocks (the paper uses no balancing
// loss; its experts simply run one after another), so a batch may send a handful of tokens to many blocks.  For such
// a group the matrix-core contractions after the selection would read the block's rows of V or K to use the few
// dozen that the group's tokens selected, and run whole tiles for a few rows.  Groups of at most `small_rows` tokens
// are therefore left out of those contractions (the tile schedule lists them last; see TokenSched) and handled here
// pair by pair:
//   forward   out[t, :]      += sum over the token's selected neurons j of the block of act * V[j, :]        (Eq. 4)
//   backward  ds[t, i]        = act > 0 ? dOut[t, :] . V[j, :] : 0;   dh[t, :] += sum ds * K[j, :]
//             dV[j, :], dK[j, :] of the block's touched neurons, the group's tokens summed in ascending order
// (Section 3.1, last paragraph).  The key scores of a small group still come from the score contraction: every
// neuron of a routed block has to be scored whatever the group's size (Eq. 6).
// A pair moves one row of d elements, so these kernels are bound by latency rather than by arithmetic: the work of
// one entry is spread over many waves (column chunks of 512 elements across workgroups, pairs across the waves of a
// workgroup), every sum in an order that the launch alone fixes.
// A token's row of out or dh is the sum of its entries' rows; the kernel that forms it (token_rows_body) takes an entry of
// a large group from `part` and works through the pairs of the others itself, so a small group costs the forward no
// launch of its own and its part of the row stays in fp32.  The backward's own small-group work shares launches with
// other work that does not depend on it: the activation gradients with the compaction of the touched list, the dV / dK
// rows with the dh rows.  (A launch that finds nothing to do costs 4 us: four of them were a fifth of a 2048-token
// step at d = 1024.)
// The entries of the small groups are listed once per dispatch (small_lists_body); worker x of a launch takes the
// entries x, x + workers, ... of that list, so consecutive workgroups, which go to the XCDs in turn, hold
// consecutive entries and every XCD gets its share of the memory traffic.
#pragma once
#include "common.h"
#include "select.h"

#ifndef MEFT_SMALL_ROWS
#define MEFT_SMALL_ROWS 16
#endif

namespace meft {

constexpr int kSmallRowChunk = 16;  // neurons per workgroup of the dV / dK kernel
constexpr int kSmallRowsMax = 16;   // upper limit of small_rows (size of that kernel's tables)
constexpr int kSmallRows = MEFT_SMALL_ROWS;   // a group of at most this many tokens is small; 0 switches the path off
constexpr int kSmallCols = 512;     // elements of a row that one wave covers in one step: 64 lanes x 8
constexpr int kSmallPairSplit = 8;  // workgroups that share the pairs of one entry in small_ds_body
constexpr int kSmallSlot = (int)0x80000000;   // in slot_of_ent: the entry's group is small
static_assert(kSmallRows >= 0 && kSmallRows <= kSmallRowsMax, "the tables of small_dvdk_body hold kSmallRowsMax tokens");

// acc += cf * eight bf16 values
__device__ __forceinline__ void fma8_bf16(float cf, u32x4 x, float (&acc)[8]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    acc[2 * i] = fmaf(cf, __uint_as_float(x[i] << 16), acc[2 * i]);
    acc[2 * i + 1] = fmaf(cf, __uint_as_float(x[i] & 0xFFFF0000u), acc[2 * i + 1]);
  }
}

// exclusive scan of one 0 / 1 flag per thread over a workgroup of whole waves (at most 256 threads)
__device__ __forceinline__ int flag_excl_scan(bool v, int* s_wave /*[4]*/, int& total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const unsigned long long m = __ballot(v);
  if (lane == 0) s_wave[w] = __popcll(m);
  __syncthreads();
  int base = 0, tot = 0;
  for (int i = 0; i < nw; ++i) { const int x = s_wave[i]; base += i < w ? x : 0; tot += x; }
  total = tot;
  __syncthreads();
  return base + __popcll(m & ((1ull << lane) - 1ull));
}

// Positions p (ascending) of the pairs of one token whose neuron lies in block g, into s_list; returns their number.
// `it` = the token's idx row (any order), k entries.  s_w: 4 ints of scratch.  Called by all the threads.
__device__ __forceinline__ int collect_block_pairs(const int32_t* __restrict__ it, int k, int N, int bs, int g,
                                                   int* s_list, int* s_w) {
  int n = 0;
  for (int p0 = 0; p0 < k; p0 += blockDim.x) {
    const int p = p0 + (int)threadIdx.x;
    const bool hit = p < k && clampi(it[p], 0, N - 1) / bs == g;
    int tot;
    const int pos = flag_excl_scan(hit, s_w, tot);
    if (hit) s_list[n + pos] = p;
    n += tot;
  }
  __syncthreads();
  return n;
}

// The small groups of a dispatch and their entries, in group order: small_grp[0 .. small_cnt[1]) = groups of 1 to
// small_rows tokens, small_ent[0 .. small_cnt[0]) = (group, slot) of their entries.  The kernels below walk these
// lists, so that their launches need not cover every (group, token) position.  n_groups <= 1024; executed by one
// whole workgroup of 1024 threads (s_w: 16 ints of scratch).
__device__ __forceinline__ void small_lists_body(int rows, int s0, int n_groups, int small_rows, int2* __restrict__ small_ent, int32_t* __restrict__ small_grp,
                                                 int32_t* __restrict__ small_cnt, int* s_w) {
  // rows, s0: number of entries and first slot of group threadIdx.x (0 rows beyond n_groups)
  const int tid = threadIdx.x;
  const bool sm = rows > 0 && rows <= small_rows;
  int tot_e, tot_g;
  const int eo = block_excl_scan_1024(sm ? rows : 0, s_w, tot_e);
  const int go = block_excl_scan_1024(sm ? 1 : 0, s_w, tot_g);
  if (sm) {
    small_grp[go] = tid;
    for (int i = 0; i < rows; ++i) small_ent[eo + i] = make_int2(tid, s0 + i);
  }
  if (tid == 0) { small_cnt[0] = tot_e; small_cnt[1] = tot_g; }
}

__global__ __launch_bounds__(1024) void small_lists_kernel(const int32_t* __restrict__ group_off, int n_groups,
                                                           int small_rows, int2* __restrict__ small_ent,
                                                           int32_t* __restrict__ small_grp,
                                                           int32_t* __restrict__ small_cnt) {
  __shared__ int s_w[16];
  const int tid = threadIdx.x, s0 = tid < n_groups ? group_off[tid] : 0;
  small_lists_body(tid < n_groups ? group_off[tid + 1] - s0 : 0, s0, n_groups, small_rows, small_ent, small_grp, small_cnt,
                   s_w);
}

// The rows of one token: row[t, :] = sum over its entries of large groups of part[slot, :] (bf16), plus sum over its
// pairs of small groups of coef[t, p] * W[j, :] (W = V, coef = act: out; W = K, coef = ds: dh); fp32 sums, large groups in
// ascending block order first, then the pairs in list order.  One workgroup per token, thread tid owns the columns
// (tid + v * blockDim.x) * 8.  s_list: min(k, kTokenRowsPairs) pairs, s_blk: kTokenRowsBlocks ints.  The pairs are listed
// kTokenRowsPairs positions at a time: a list of all of a large top_k (64 KB at 8192) leaves a compute unit too few
// workgroups for what is otherwise a stream (out rows of 4096 tokens x 8 entries x 4096: 61 us without the list, 104 with).
constexpr int kTokenRowsBlocks = 64, kTokenRowsPairs = 1024;

struct TokenRows {
  const uint16_t* part;
  const int32_t *sblk, *slot_of_ent, *idx;
  const float* coef;
  const bf16_t* W;
  int d, e, k, N, bs;
  bf16_t* out;
  bool past_l2;   // how the partial rows are read (rows_past_l2)
};

// the token's blocks whose groups are small, into s_blk
__device__ __forceinline__ void collect_small_blocks(const TokenRows& a, int t, int* s_blk) {
  for (int q = threadIdx.x; q < min(a.e, kTokenRowsBlocks); q += blockDim.x)
    s_blk[q] = a.slot_of_ent[(size_t)t * a.e + q] < 0 ? a.sblk[(size_t)t * a.e + q] : -1;
  __syncthreads();
}

// the token's pairs of small groups among its positions first .. first + kTokenRowsPairs - 1, ascending, into s_list: neuron,
// coefficient.  (The first scan's barriers keep the list until everyone has read the one before.)
__device__ __forceinline__ int collect_small_pairs(const TokenRows& a, int t, int first, int2* s_list, const int* s_blk,
                                                   int* s_w) {
  const int32_t* it = a.idx + (size_t)t * a.k;
  const float* ct = a.coef + (size_t)t * a.k;
  const int nb = min(a.e, kTokenRowsBlocks), end = min(a.k, first + kTokenRowsPairs);
  int n = 0;
  for (int p0 = first; p0 < end; p0 += blockDim.x) {
    const int p = p0 + (int)threadIdx.x;
    bool hit = false;
    int j = 0;
    float cf = 0.f;
    if (p < end) {
      j = clampi(it[p], 0, a.N - 1);
      cf = ct[p];
      const int b = j / a.bs;
      for (int q = 0; q < nb; ++q) hit |= s_blk[q] == b;
      for (int q = nb; q < a.e; ++q)
        hit |= a.sblk[(size_t)t * a.e + q] == b && a.slot_of_ent[(size_t)t * a.e + q] < 0;
    }
    int tot;
    const int pos = flag_excl_scan(hit, s_w, tot);
    if (hit) s_list[n + pos] = make_int2(j, __float_as_int(cf));
    n += tot;
  }
  __syncthreads();
  return n;
}

template <int NV>
__device__ __forceinline__ void token_rows_body(const TokenRows& a, int t, int2* s_list, int* s_blk, int* s_w) {
  const int tid = threadIdx.x, nthr = blockDim.x, d = a.d;
  float acc[NV][8];
#pragma unroll
  for (int v = 0; v < NV; ++v)
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[v][c] = 0.f;
  bool small = false;
  auto sum_partial = [&](auto past_l2) {
    for (int q = 0; q < a.e; ++q) {
      if (a.sblk[(size_t)t * a.e + q] < 0) continue;
      const int slot = a.slot_of_ent[(size_t)t * a.e + q];
      if (slot < 0) { small = true; continue; }
      const bf16_t* row = reinterpret_cast<const bf16_t*>(a.part) + (size_t)slot * d;
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const int col = (tid + v * nthr) * 8;
        if (col < d) {
          float x[8];
          if constexpr (decltype(past_l2)::value) Vec8<bf16_t>::load_once(row + col, x);
          else Vec8<bf16_t>::load(row + col, x);
#pragma unroll
          for (int c = 0; c < 8; ++c) acc[v][c] += x[c];
        }
      }
    }
  };
  if (a.past_l2) sum_partial(std::true_type{});
  else sum_partial(std::false_type{});
  if (small) {   // the same in every thread
    collect_small_blocks(a, t, s_blk);
    constexpr int U = NV == 1 ? 16 : NV == 2 ? 8 : NV == 4 ? 4 : 2;   // rows in flight
    for (int p0 = 0; p0 < a.k; p0 += kTokenRowsPairs) {
      const int n = collect_small_pairs(a, t, p0, s_list, s_blk, s_w);
      for (int q0 = 0; q0 < n; q0 += U) {
        u32x4 x[U][NV];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const bf16_t* row = a.W + (size_t)s_list[min(q0 + u, n - 1)].x * d;
#pragma unroll
          for (int v = 0; v < NV; ++v) {
            const int col = (tid + v * nthr) * 8;
            if (col < d) x[u][v] = *reinterpret_cast<const u32x4*>(row + col);
          }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (q0 + u < n) {
            const float cf = __int_as_float(s_list[q0 + u].y);
#pragma unroll
            for (int v = 0; v < NV; ++v)
              if ((tid + v * nthr) * 8 < d) fma8_bf16(cf, x[u][v], acc[v]);
          }
        }
      }
    }
  }
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int col = (tid + v * nthr) * 8;
    if (col < d) Vec8<bf16_t>::store(a.out + (size_t)t * d + col, acc[v]);
  }
}

// The same for few tokens: a workgroup of four waves per (token, 512 columns); the entries and the pairs are dealt to the
// waves, whose sums are added in wave order.
__device__ __forceinline__ void token_rows_split_body(const TokenRows& a, int t, int chunk, int2* s_list, int* s_blk,
                                                      int* s_w, float (&s_red)[3][kSmallCols]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, d = a.d;
  const int col = chunk * kSmallCols + lane * 8;
  const bool live = col < d;
  float acc[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) acc[c] = 0.f;
  bool small = false;
  for (int q = 0; q < a.e; ++q) {
    if (a.sblk[(size_t)t * a.e + q] < 0) continue;
    const int slot = a.slot_of_ent[(size_t)t * a.e + q];
    if (slot < 0) { small = true; continue; }
    if ((q & 3) == wave && live) {
      float x[8];
      Vec8<bf16_t>::load(reinterpret_cast<const bf16_t*>(a.part) + (size_t)slot * d + col, x);
#pragma unroll
      for (int c = 0; c < 8; ++c) acc[c] += x[c];
    }
  }
  if (small) {
    collect_small_blocks(a, t, s_blk);
    constexpr int U = 8;
    int before = 0;   // pairs of the lists before: pair number i of all goes to wave i % 4
    for (int p0 = 0; p0 < a.k; p0 += kTokenRowsPairs) {
      const int n = collect_small_pairs(a, t, p0, s_list, s_blk, s_w);
      for (int q0 = (wave - before) & 3; q0 < n && live; q0 += 4 * U) {
        u32x4 x[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
          x[u] = *reinterpret_cast<const u32x4*>(a.W + (size_t)s_list[min(q0 + 4 * u, n - 1)].x * d + col);
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (q0 + 4 * u < n) fma8_bf16(__int_as_float(s_list[q0 + 4 * u].y), x[u], acc);
      }
      before += n;
    }
  }
  if (wave > 0) Vec8<float>::store(&s_red[wave - 1][lane * 8], acc);
  __syncthreads();
  if (wave == 0 && live) {
#pragma unroll
    for (int w = 0; w < 3; ++w)
#pragma unroll
      for (int c = 0; c < 8; ++c) acc[c] += s_red[w][lane * 8 + c];
    Vec8<bf16_t>::store(a.out + (size_t)t * d + col, acc);
  }
}

// backward: ds32[t * k + p] = act > 0 ? dOut[t, :] . V[j, :] : 0 for the pairs of the entry; one wave per pair, the
// entry's pairs dealt to the 4 * kSmallPairSplit waves of the workers with the same wx and wy = 0 .. kSmallPairSplit - 1.
// s_list: k ints.
__device__ __forceinline__ void small_ds_body(int wx, int nx, int wy, int* s_list, int* s_w, const bf16_t* __restrict__ V, const bf16_t* __restrict__ dOut,
                                                       const int32_t* __restrict__ idx, const float* __restrict__ act,
                                                       const int2* __restrict__ small_ent,
                                                       const int32_t* __restrict__ small_cnt,
                                                       const int32_t* __restrict__ tok_of_slot, int d, int k, int N,
                                                       int bs, float* __restrict__ ds32) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n_ent = small_cnt[0];
  for (int e = wx; e < n_ent; e += nx) {
    const int g = small_ent[e].x, t = tok_of_slot[small_ent[e].y];
    const int32_t* it = idx + (size_t)t * k;
    const float* at = act + (size_t)t * k;
    const int n = collect_block_pairs(it, k, N, bs, g, s_list, s_w);
    const bf16_t* grow = dOut + (size_t)t * d;
    for (int q = wy * 4 + wave; q < n; q += 4 * kSmallPairSplit) {
      const int p = s_list[q];
      const bf16_t* vrow = V + (size_t)clampi(it[p], 0, N - 1) * d;
      float dot = 0.f;
#pragma unroll 4
      for (int col = lane * 8; col < d; col += kSmallCols) {
        float x[8], y[8];
        Vec8<bf16_t>::load(vrow + col, x);
        Vec8<bf16_t>::load(grow + col, y);
#pragma unroll
        for (int c = 0; c < 8; ++c) dot = fmaf(x[c], y[c], dot);
      }
      dot = wave_sum(dot);
      if (lane == 0) ds32[(size_t)t * k + p] = at[p] > 0.f ? dot : 0.f;
    }
    __syncthreads();   // s_list is reused by the next entry
  }
}

// backward: dV and dK rows of a small group's block.  Only this group's tokens select neurons of its block, so the
// touched rows of the block are exactly the rows some token of the group selected.  The chunk of kSmallRowChunk
// neurons is the fast launch index (wx), so that the chunks of one group, whose work is alike, go to the
// XCDs in turn whatever the sizes of the groups.  Per (group, chunk): tables in LDS say which tokens of the group
// select each neuron of the chunk, with which activation and activation gradient; the (selected neuron, 512 columns)
// pieces are dealt to the four waves, and a neuron's rows are summed over the group's tokens in ascending slot
// (= token) order.
__device__ __forceinline__ void small_dvdk_piece(const bf16_t* __restrict__ h, const bf16_t* __restrict__ dOut,
                                                 const int* tok, const float* a, const float* s, int rows, int d,
                                                 int col, float (&aK)[8], float (&aV)[8]) {
#pragma unroll
  for (int c = 0; c < 8; ++c) { aK[c] = 0.f; aV[c] = 0.f; }
  for (int i = 0; i < rows; ++i) {
    const int t = tok[i];
    if (t < 0) continue;
    float xg[8], xh[8];
    Vec8<bf16_t>::load(dOut + (size_t)t * d + col, xg);
    Vec8<bf16_t>::load(h + (size_t)t * d + col, xh);
    const float av = a[i], sv = s[i];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      aV[c] = fmaf(av, xg[c], aV[c]);
      aK[c] = fmaf(sv, xh[c], aK[c]);
    }
  }
}

__device__ __forceinline__ void small_dvdk_body(int wx, int wy, int ny, const bf16_t* __restrict__ h, const bf16_t* __restrict__ dOut,
                                                         const int32_t* __restrict__ idx, const float* __restrict__ act,
                                                         const float* __restrict__ ds32,
                                                         const int32_t* __restrict__ small_grp,
                                                         const int32_t* __restrict__ small_cnt,
                                                         const int32_t* __restrict__ group_off,
                                                         const int32_t* __restrict__ tok_of_slot, int d, int k, int N,
                                                         int bs, bf16_t* __restrict__ dK, bf16_t* __restrict__ dV) {
  __shared__ int s_tok[kSmallRowChunk][kSmallRowsMax];     // token that selects the neuron, or -1
  __shared__ float s_a[kSmallRowChunk][kSmallRowsMax];     // its activation
  __shared__ float s_s[kSmallRowChunk][kSmallRowsMax];     // its activation gradient
  __shared__ int s_rows[kSmallRowChunk];                   // the selected neurons of the chunk, ascending
  __shared__ int s_nrows;
  static_assert(kSmallRowChunk <= 64, "one lane of the first wave per neuron of the chunk");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r0 = wx * kSmallRowChunk;   // first neuron of the chunk, inside the block
  const int n_grp = small_cnt[1];
  for (int e = wy; e < n_grp; e += ny) {
    const int g = small_grp[e];
    const int slot0 = group_off[g], rows = min(group_off[g + 1] - slot0, kSmallRowsMax);   // (at most small_rows)
    for (int z = tid; z < kSmallRowChunk * kSmallRowsMax; z += 256) (&s_tok[0][0])[z] = -1;
    __syncthreads();
    // the group's rows * k pairs, four per thread and step, loads first
    const int n_pairs = rows * k;
    for (int z0 = 0; z0 < n_pairs; z0 += 4 * 256) {
      int ii[4], pp[4], tt[4], jj[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int z = z0 + u * 256 + tid;
        ii[u] = z < n_pairs ? z / k : -1;
        pp[u] = z - ii[u] * k;
        tt[u] = ii[u] >= 0 ? tok_of_slot[slot0 + ii[u]] : 0;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) jj[u] = ii[u] >= 0 ? clampi(idx[(size_t)tt[u] * k + pp[u]], 0, N - 1) : -1;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int r = jj[u] - g * bs - r0;
        if (jj[u] >= 0 && jj[u] / bs == g && r >= 0 && r < kSmallRowChunk) {   // ids are distinct inside a token: one writer per cell
          s_tok[r][ii[u]] = tt[u];
          s_a[r][ii[u]] = act[(size_t)tt[u] * k + pp[u]];
          s_s[r][ii[u]] = ds32[(size_t)tt[u] * k + pp[u]];
        }
      }
    }
    __syncthreads();
    if (wave == 0) {
      bool any = false;
      if (lane < kSmallRowChunk)
        for (int i = 0; i < rows; ++i) any |= s_tok[lane][i] >= 0;
      const unsigned long long m = __ballot(any);
      if (any) s_rows[__popcll(m & ((1ull << lane) - 1ull))] = lane;
      if (lane == 0) s_nrows = __popcll(m);
    }
    __syncthreads();
    const int cpr = (d + kSmallCols - 1) / kSmallCols;   // column pieces per row
    const int n_items = s_nrows * cpr;
    int it = wave;
    for (; it + 4 < n_items; it += 8) {   // two pieces at a time
      const int z0 = it / cpr, z1 = (it + 4) / cpr;
      const int r_0 = s_rows[z0], r_1 = s_rows[z1];
      const int c_0 = (it - z0 * cpr) * kSmallCols + lane * 8, c_1 = (it + 4 - z1 * cpr) * kSmallCols + lane * 8;
      float k0[8], v0[8], k1[8], v1[8];
      if (c_0 < d) small_dvdk_piece(h, dOut, s_tok[r_0], s_a[r_0], s_s[r_0], rows, d, c_0, k0, v0);
      if (c_1 < d) small_dvdk_piece(h, dOut, s_tok[r_1], s_a[r_1], s_s[r_1], rows, d, c_1, k1, v1);
      const size_t j0 = (size_t)g * bs + r0 + r_0, j1 = (size_t)g * bs + r0 + r_1;
      if (c_0 < d) { Vec8<bf16_t>::store(dV + j0 * d + c_0, v0); Vec8<bf16_t>::store(dK + j0 * d + c_0, k0); }
      if (c_1 < d) { Vec8<bf16_t>::store(dV + j1 * d + c_1, v1); Vec8<bf16_t>::store(dK + j1 * d + c_1, k1); }
    }
    for (; it < n_items; it += 4) {
      const int z0 = it / cpr, r_0 = s_rows[z0];
      const int c_0 = (it - z0 * cpr) * kSmallCols + lane * 8;
      if (c_0 >= d) continue;
      float k0[8], v0[8];
      small_dvdk_piece(h, dOut, s_tok[r_0], s_a[r_0], s_s[r_0], rows, d, c_0, k0, v0);
      const size_t j0 = (size_t)g * bs + r0 + r_0;
      Vec8<bf16_t>::store(dV + j0 * d + c_0, v0);
      Vec8<bf16_t>::store(dK + j0 * d + c_0, k0);
    }
    __syncthreads();   // the tables are reused by the next group
  }
}

}  // namespace meft
