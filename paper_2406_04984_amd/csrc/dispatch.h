// (token, block) dispatch: the grouping of the T * top_e (token, block) entries by block that the grouped GEMMs work
// from.  Entry i = t * top_e + q holds block sblk[i] (or -1), the blocks of a token ascending; slots are the entries
// sorted by block, entries of one block in ascending entry (= token) order:
//   perm[slot] = entry, group_off[b] = first slot of block b, cnt[b] = its entries, tile_off = prefix of
//   ceil(cnt / BM), and on the matrix-core path tok_of_slot, slot_of_ent and the per-XCD tile schedule.
// slot_of_ent carries kSmallSlot where the entry's group is one of at most small_rows tokens (small_groups.h).
//
// Small dispatches (dispatch_one_form) take one launch: a workgroup per block looks through all the entries (they come out of L2,
// and a launch costs more) and places its own, and one more counts the entries of all blocks, writes the tables and deals the
// groups to the XCDs.  Two launches / one: 2048 tokens x 4, 64 blocks 21.8 -> 11.2 us; 8192 x 4, 64 blocks 24 -> 14; 4096 x 8, 256
// blocks 30 -> 18 (of either about half by the faster tables).  At the limits, whole forward of a layer with d 64: 16384 x 4, 64
// blocks 105.2 -> 99.8, 128 blocks 116.3 -> 105.4; beyond them 16384 x 8, 16 blocks 114.2 -> 126.1.
// Beyond that, up to 1024 blocks and 2^20 entries, it takes two launches over chunks of whole tokens, at most 1024 entries each:
//   dispatch_count   sorts every token's blocks, counts the entries of every block per chunk, and clears what the
//                    forward or backward needs cleared;
//   dispatch_place   every workgroup adds the chunk counts up for itself (a few thousand integers out of L2 cost less
//                    than a launch) and places its chunk's entries, while one more workgroup writes the tables and
//                    deals the groups to the XCDs, which is a serial chain.
// Against four launches (sort, count, one workgroup that scans and deals, place): 41 -> 24 us at 8192 x 4 entries and 64
// blocks, 67 -> 30 us at 4096 x 8 and 256.  Where the chunk counts are too many for every workgroup to add up (more than
// kDispScanMax), one workgroup does it in a launch of its own in between.
// The rank of an entry inside its wave comes from ballots over the distinct blocks of the wave, the rest from prefix
// sums, so the order is the entry order and nothing depends on the timing of atomics.
// (Shapes beyond these limits use count_blocks / fill_groups / slot_maps / build_sched, which scan the entries
// once per block.)
#pragma once
#include "gemm_mfma.h"
#include "select.h"
#include "small_groups.h"

namespace meft {

constexpr int kDispMaxBlocks = 1024;    // LDS: 16 waves x n_blocks counters
constexpr int kDispMaxEntries = 1 << 20;   // at most 2045 chunks (of 513 entries at top_e 513)
constexpr int kDispScanBlocks = 512;    // dispatch_place adds up the chunk counts itself up to this many blocks
constexpr int kDispScanMax = 32768;     // and this many counts

constexpr int kDispOneTokens = 16 * 1024;   // one launch: tokens (sixteen per thread)
constexpr int kDispOneEntries = 1 << 16;    // entries, which one workgroup counts
constexpr int kDispOneWork = 1 << 23;       // entries x blocks
constexpr int kDispOneShare = 3584;         // and, beyond kDispFewTokens tokens, entries per block
constexpr int kDispFewTokens = 4096;        // more tokens, and at least 256 for each block (at most 64 blocks, then): kFew
// Which form of dispatch_one_kernel: 0 none (two launches), 1 kFew, 2 the other.
// Forwards without the value sum of layers with d 64 (us; two launches / one, without and with kFew): 16384 tokens x 1, one block
// 60.2 / 69.6 / 59.3; x 4, 4 blocks 71.0 / 82.6 / 74.7; x 4, 16 blocks 75.6 / 79.9 / 76.6; 8192 x 8, 16 blocks 53.9 / 55.8 / 55.0;
// 8192 x 4, 8 blocks 46.6 / 46.8 / 45.4; 6000 x 8, 16 blocks 44.8 / 43.8 / 44.1; 16384 x 4, 32 blocks 79.3 / 79.7 / 78.4; and with
// Zipf-popular blocks 16384 x 4, 32 blocks 79.3 / 84.3 / 79.2; 8192 x 8, 24 blocks 55.4 / 58.6 / 55.6; 6000 x 4, 8 blocks 40.2 /
// 39.8 / 38.0; 16384 x 4, 64 blocks 84.3 / 85.5 / 81.6 (with blocks alike 85.0 / 80.3 / 80.9).
inline int dispatch_one_form(int n_tok, int e, int n_blocks) {
  const long long n_ent = (long long)n_tok * e;
  if (n_blocks > kDispMaxBlocks || n_tok > kDispOneTokens || n_ent > kDispOneEntries || n_ent * n_blocks > kDispOneWork) return 0;
  if (n_tok <= kDispFewTokens) return 2;
  if (n_ent > (long long)kDispOneShare * n_blocks) return 0;
  return n_blocks * 256 <= n_tok ? 1 : 2;
}

// Rank of this lane's entry among the entries of the same block in its wave, in lane (= entry) order; lane
// `leader of the block` also writes the block's count in the wave to row[block] (row zeroed by the caller).
__device__ __forceinline__ int wave_block_ranks(int b, int* row) {
  const int lane = threadIdx.x & 63;
  int rank = 0;
  unsigned long long todo = __ballot(b >= 0);
  while (todo) {   // wave-uniform: one round per distinct block of the wave
    const int leader = __ffsll(todo) - 1;
    const int b0 = __builtin_amdgcn_readlane(b, leader);
    const unsigned long long m = __ballot(b == b0);
    if (b == b0) rank = __popcll(m & ((1ull << lane) - 1ull));
    if (lane == leader) row[b0] = __popcll(m);
    todo &= ~m;
  }
  return rank;
}

// pass 1: H[chunk][b] = entries of block b in the chunk.  kSort: `in` holds the token's blocks in any order, ids are
// clamped and written to sblk ascending; otherwise `in` is sblk (-1: no entry).  `epc` entries per chunk (whole
// tokens).  Also zeroes clear[0 .. clear_words).  Dynamic LDS: 16 * n_blocks ints.
template <bool kSort>
__global__ __launch_bounds__(1024) void dispatch_count_kernel(const int32_t* __restrict__ in, int n_ent, int e, int epc,
                                                              int n_blocks, int32_t* __restrict__ sblk,
                                                              int32_t* __restrict__ H, int32_t* __restrict__ clear,
                                                              size_t clear_words) {
  extern __shared__ int s_cnt[];   // [16 waves][n_blocks]
  __shared__ int s_in[kSort ? 1024 : 1], s_out[kSort ? 1024 : 1];
  const int tid = threadIdx.x, w = tid >> 6, c = blockIdx.x;
  for (size_t i = (size_t)c * 1024 + tid; i < clear_words; i += (size_t)gridDim.x * 1024) clear[i] = 0;
  for (int i = tid; i < 16 * n_blocks; i += 1024) s_cnt[i] = 0;
  const int i = c * epc + tid;
  const bool live = tid < epc && i < n_ent;
  int b = live ? in[i] : -1;
  if constexpr (kSort) {
    b = live ? clampi(b, 0, n_blocks - 1) : -1;
    s_in[tid] = b;
    __syncthreads();
    if (live) {
      const int q = tid % e, base = tid - q;
      int r = 0;
      for (int z = 0; z < e; ++z) {
        const int bz = s_in[base + z];
        r += (bz < b || (bz == b && z < q)) ? 1 : 0;
      }
      s_out[base + r] = b;
    }
    __syncthreads();
    if (live) { b = s_out[tid]; sblk[i] = b; }
  } else {
    b = (unsigned)b < (unsigned)n_blocks ? b : -1;
    __syncthreads();
  }
  wave_block_ranks(b, s_cnt + w * n_blocks);
  __syncthreads();
  for (int bb = tid; bb < n_blocks; bb += 1024) {
    int run = 0;
#pragma unroll
    for (int ww = 0; ww < 16; ++ww) run += s_cnt[ww * n_blocks + bb];
    H[(size_t)c * n_blocks + bb] = run;
  }
}

// What the dispatch leaves besides perm and the slot maps.
struct DispatchTables {
  int32_t *cnt, *group_off, *tile_off;
  int BM;                 // rows per tile of tile_off
  int cap;                // tile schedule: entries per XCD
  int4* grp;              // nullptr: no tile schedule
  int2* tiles;
  int* len;
  int small_rows;
  int2* small_ent;        // nullptr: no lists of small groups
  int32_t *small_grp, *small_cnt;
};

// Entries of block tid (0 beyond n_blocks) -> all the tables; with pad_tok also `pad` valid entries behind the last slot of
// tok_of_slot.  Executed by one whole workgroup of 1024 threads, once per launch, so it is written for short code rather than
// few instructions: what runs once waits for its instructions to come from memory.
__device__ __forceinline__ void dispatch_tables(const DispatchTables& t, int rows, int n_blocks, int* s_w, int32_t* pad_tok,
                                                int pad) {
  const int tid = threadIdx.x;
  int all_g, all_t;
  const int go = block_excl_scan_1024(rows, s_w, all_g);
  if (tid < n_blocks) { t.cnt[tid] = rows; t.group_off[tid] = go; }
  if (tid == 0) t.group_off[n_blocks] = all_g;
  if (t.grp == nullptr) {   // (the contractions on a tile schedule do not use it)
    const int to = block_excl_scan_1024((rows + t.BM - 1) / t.BM, s_w, all_t);
    if (tid < n_blocks) t.tile_off[tid] = to;
    if (tid == 0) t.tile_off[n_blocks] = all_t;
  }
  if (pad_tok != nullptr && tid < pad) pad_tok[all_g + tid] = 0;   // (entries of block -1 have no slot)
  if (t.small_ent != nullptr) {
    small_lists_body(rows, go, n_blocks, t.small_rows, t.small_ent, t.small_grp, t.small_cnt, s_w);
  }
  if (t.grp != nullptr) build_sched_body(rows, go, n_blocks, t.cap, t.grp, t.tiles, t.len, t.small_rows);   // (no barrier after it)
}

// Between the passes where the counts are many, one workgroup: H[chunk][b] becomes the number of entries of block b in
// the chunks before; the tables.
__global__ __launch_bounds__(1024) void dispatch_scan_kernel(int32_t* __restrict__ H, int n_chunks, int n_blocks,
                                                             DispatchTables t) {
  __shared__ int s_w[16];
  const int tid = threadIdx.x;   // = block, n_blocks <= 1024
  int tot = 0;
  if (tid < n_blocks) {
    // sixteen independent loads at a time: the serial part is the additions, not the memory latency
    for (int c0 = 0; c0 < n_chunks; c0 += 16) {
      int v[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) v[j] = c0 + j < n_chunks ? H[(size_t)(c0 + j) * n_blocks + tid] : 0;
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        if (c0 + j < n_chunks) H[(size_t)(c0 + j) * n_blocks + tid] = tot;
        tot += v[j];
      }
    }
  }
  dispatch_tables(t, tot, n_blocks, s_w, nullptr, 0);
}

// pass 2: perm, and with tok_of_slot != nullptr the slot maps (tok_of_slot padded by `pad` valid entries).
// kScan: H holds the chunk counts, every workgroup adds them up, and workgroup number n_chunks writes the tables; lg =
// log2 of the power of two at or above n_blocks.  Otherwise H and the tables come from dispatch_scan_kernel.
// Dynamic LDS: 16 * n_blocks ints.
template <bool kScan>
__global__ __launch_bounds__(1024) void dispatch_place_kernel(const int32_t* __restrict__ sblk, int n_ent, int e, int epc,
                                                              int n_blocks, int lg, int n_chunks,
                                                              const int32_t* __restrict__ H, DispatchTables tab,
                                                              int32_t* __restrict__ perm,
                                                              int32_t* __restrict__ tok_of_slot,
                                                              int32_t* __restrict__ slot_of_ent, int pad) {
  extern __shared__ int s_cnt[];   // [16 waves][n_blocks]
  __shared__ int s_w[16];
  __shared__ int s_tot[kScan ? kDispScanBlocks : 1], s_first[kScan ? kDispScanBlocks : 1];
  const int tid = threadIdx.x, w = tid >> 6, c = blockIdx.x;
  const int i = c * epc + tid;
  int b = c < n_chunks && tid < epc && i < n_ent ? sblk[i] : -1;
  b = (unsigned)b < (unsigned)n_blocks ? b : -1;
  if constexpr (kScan) {
    if (tid < n_blocks) { s_tot[tid] = 0; s_first[tid] = 0; }
    __syncthreads();
    const int bb = tid & ((1 << lg) - 1), parts = 1024 >> lg;
    if (bb < n_blocks) {
      int tot = 0, before = 0;
      for (int ch = tid >> lg; ch < n_chunks; ch += parts) {
        const int v = H[(size_t)ch * n_blocks + bb];
        tot += v;
        before += ch < c ? v : 0;
      }
      atomicAdd(&s_tot[bb], tot);
      atomicAdd(&s_first[bb], before);
    }
    __syncthreads();
    const int rows = tid < n_blocks ? s_tot[tid] : 0;
    if (c == n_chunks) {
      dispatch_tables(tab, rows, n_blocks, s_w, tok_of_slot, pad);
      return;
    }
    int all;
    const int go = block_excl_scan_1024(rows, s_w, all);
    if (tid < n_blocks) s_first[tid] += go;
  }
  for (int z = tid; z < 16 * n_blocks; z += 1024) s_cnt[z] = 0;
  __syncthreads();
  const int rank = wave_block_ranks(b, s_cnt + w * n_blocks);
  __syncthreads();
  // per block: first slot of wave 0's entries, then the exclusive prefix over the waves
  for (int bb = tid; bb < n_blocks; bb += 1024) {
    int run;
    if constexpr (kScan) run = s_first[bb];
    else run = tab.group_off[bb] + H[(size_t)c * n_blocks + bb];
#pragma unroll
    for (int ww = 0; ww < 16; ++ww) {
      const int t = s_cnt[ww * n_blocks + bb];
      s_cnt[ww * n_blocks + bb] = run;
      run += t;
    }
  }
  __syncthreads();
  if (b >= 0) {
    const int slot = s_cnt[w * n_blocks + b] + rank;
    perm[slot] = i;
    if (tok_of_slot != nullptr) {
      int rows;
      if constexpr (kScan) rows = s_tot[b];
      else rows = tab.cnt[b];
      tok_of_slot[slot] = i / e;
      slot_of_ent[i] = rows <= tab.small_rows ? (slot | kSmallSlot) : slot;
    }
  }
  if (!kScan && tok_of_slot != nullptr && c == 0 && tid < pad) tok_of_slot[tab.group_off[n_blocks] + tid] = 0;
}

// The whole dispatch in one launch of n_blocks + 1 workgroups.  kSort: `in` holds the token's blocks in any order, ids are
// clamped, and sblk is written; otherwise `in` is sblk (-1: no entry).  A block that a token names twice gets two entries.
// Also zeroes clear[0 .. clear_words).
// kFew, for few blocks and many tokens, where what a workgroup does one step after the other is all there is: n_blocks * parts + 1
// workgroups, part p of a block's placing the tokens p * 1024 .. of every parts * 1024 (all of them count the block's); several
// steps' loads on their way together; several counters per block.  (The other form is as short as it was: code that runs once
// waits for its instructions to come from memory; with all of this it took 0.7 us more at 2048 tokens x 4, 64 blocks.)
template <bool kSort, bool kFew>
__global__ __launch_bounds__(1024) void dispatch_one_kernel(const int32_t* __restrict__ in, int n_tok, int e, int n_blocks,
                                                            DispatchTables tab, int32_t* __restrict__ sblk,
                                                            int32_t* __restrict__ perm, int32_t* __restrict__ tok_of_slot,
                                                            int32_t* __restrict__ slot_of_ent, int pad,
                                                            int32_t* __restrict__ clear, size_t clear_words) {
  extern __shared__ int s_one[];   // [iterations][1024]: per token, blocks below b << 16 | entries of b;  [iterations * 16]
  __shared__ int s_w[16];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int n_ent = n_tok * e, n_iter = (n_tok + 1023) >> 10;
  for (size_t i = (size_t)blockIdx.x * 1024 + tid; i < clear_words; i += (size_t)gridDim.x * 1024) clear[i] = 0;
  if (blockIdx.x == 0) {   // (first, as it takes longest)
    // kFew: kCopies counters per block, which the lanes of a wave share out among them (adding to one word is done lane by lane)
    constexpr int kCopies = kFew ? 16 : 1;
    if (tid < n_blocks * kCopies) s_one[tid] = 0;
    __syncthreads();
    for (int i0 = 0; i0 < n_ent; i0 += 8 * 1024) {   // (eight loads on their way together)
      int b[8];
#pragma unroll
      for (int z = 0; z < 8; ++z) {
        const int i = i0 + z * 1024 + tid;
        b[z] = in[min(i, n_ent - 1)];
        if constexpr (kSort) b[z] = clampi(b[z], 0, n_blocks - 1);
        b[z] = i < n_ent ? b[z] : -1;
      }
#pragma unroll
      for (int z = 0; z < 8; ++z)
        if ((unsigned)b[z] < (unsigned)n_blocks) atomicAdd(&s_one[b[z] * kCopies + lane % kCopies], 1);
    }
    __syncthreads();
    if constexpr (kFew) {
      int all = tid < n_blocks * kCopies ? s_one[tid] : 0;
#pragma unroll
      for (int z = 1; z < kCopies; z <<= 1) all += __shfl_xor(all, z, kWave);
      __syncthreads();
      if (tid % kCopies == 0 && tid < n_blocks * kCopies) s_one[tid / kCopies] = all;
      __syncthreads();
    }
    dispatch_tables(tab, tid < n_blocks ? s_one[tid] : 0, n_blocks, s_w, tok_of_slot, pad);
    return;
  }
  int b = (int)blockIdx.x - 1, part = 0, parts = 1;
  if constexpr (kFew) { parts = ((int)gridDim.x - 1) / n_blocks; part = b / n_blocks; b -= part * n_blocks; }
  int* s_cnt = s_one + n_iter * 1024;
  int below = 0;   // entries of this thread's tokens that belong to blocks before b
  // (kIt iterations' loads on their way together)
  auto look = [&](auto its, int it0) {
    constexpr int kIt = decltype(its)::value;
    int lt[kIt], eq[kIt];
    const int32_t* row[kIt];
#pragma unroll
    for (int u = 0; u < kIt; ++u) {
      lt[u] = eq[u] = 0;
      row[u] = in + (size_t)min((it0 + u) * 1024 + tid, n_tok - 1) * e;
    }
#pragma unroll 4
    for (int q = 0; q < e; ++q) {
#pragma unroll
      for (int u = 0; u < kIt; ++u) {
        int x = row[u][q];
        if constexpr (kSort) x = clampi(x, 0, n_blocks - 1);
        lt[u] += (unsigned)x < (unsigned)b ? 1 : 0;
        eq[u] += x == b ? 1 : 0;
      }
    }
#pragma unroll
    for (int u = 0; u < kIt; ++u) {
      if ((it0 + u) * 1024 + tid >= n_tok) lt[u] = eq[u] = 0;
      below += lt[u];
      s_one[(it0 + u) * 1024 + tid] = lt[u] << 16 | eq[u];
      const int incl = wave_incl_scan(eq[u]);
      if (lane == 63) s_cnt[(it0 + u) * 16 + w] = incl;
    }
  };
  int it0 = 0;
  if constexpr (kFew) {
#pragma unroll 1
    for (; it0 + 4 <= n_iter; it0 += 4) look(std::integral_constant<int, 4>{}, it0);
  }
#pragma unroll 1
  for (; it0 < n_iter; ++it0) look(std::integral_constant<int, 1>{}, it0);
  int base, rows;   // entries of the blocks before, entries of this one
  block_excl_scan_1024(below, s_w, base);   // (its barriers order the counts above as well)
  const int mine = tid < n_iter * 16 ? s_cnt[tid] : 0;
  const int before = block_excl_scan_1024(mine, s_w, rows);
  if (tid < n_iter * 16) s_cnt[tid] = before;
  __syncthreads();
  const int flag = tok_of_slot != nullptr && rows <= tab.small_rows ? kSmallSlot : 0;
#pragma unroll 1
  for (int it = part; it < n_iter; it += parts) {
    const int t = it * 1024 + tid, lt = s_one[t] >> 16, eq = s_one[t] & 0xFFFF;
    const int first = base + s_cnt[it * 16 + w] + wave_incl_scan(eq) - eq;
    for (int z = 0; z < eq; ++z) {
      const int ent = t * e + lt + z, slot = first + z;
      perm[slot] = ent;
      if constexpr (kSort) sblk[ent] = b;
      if (tok_of_slot != nullptr) {
        tok_of_slot[slot] = t;
        slot_of_ent[ent] = slot | flag;
      }
    }
  }
}

}  // namespace meft
