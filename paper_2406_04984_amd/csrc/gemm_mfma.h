// Grouped bf16 GEMM core for gfx950 matrix cores, shared by every dense contraction of the layer:
//
//   C[m, n] = sum_k A(m, k) * B(k, n)          fp32 accumulation, v_mfma_f32_32x32x16_bf16
//
// Each operand is contiguous either along the contraction index or along its own index:
//   A k-contiguous (rows indexed by m) / B k-contiguous (rows indexed by n): router and key scores (Eq. 5, Eq. 6)
//     and dOut . V^T in the backward;
//   B n-contiguous (rows indexed by k): where the contraction runs over neurons or tokens while the rows of V, K,
//     dOut, h are contiguous in d: the value sum of Eq. 4, dh, dK, dV;
//   A m-contiguous (rows indexed by k): dK, dV, whose A operand is the slot-major activation matrix, read as it is.
//
// Tile 128 (m) x 256 (n) x 64 (k): 4 compute waves as 2 x 2, each wave 64 x 128 = 2 x 4 MFMA tiles, plus two or four
// loader waves that own the whole global -> LDS traffic (16 B per lane).  Ring depths kSA, kSB up to three.  Problems that fill
// 256 x 256 tiles go to gemm_wide_kernel (gemm_wide.h); here are the router, small groups, operands beyond buffer loads.
// The operands have a ring each in LDS: kSA slots of 128 x 64 for A, kSB slots of 256 x 64 for B.  (A 192-row tile
// for the token-major problems moves 22 % fewer operand bytes per flop than the 128-row one and was measured 15 %
// faster per flop, but their groups then fill a whole number of tiles worse and the step as a whole did not gain.  It
// is gone; the tile schedule has prefixes of 64 and 128 rows only.)
// LDS layouts are XOR-swizzled so that both the linear DMA writes and the fragment reads are free of bank conflicts:
//   k-contiguous operand: rows of 64 k = 8 chunks of 16 B; logical chunk c of row r sits at chunk
//     c ^ ((r >> 1) & 7); fragments are read with ds_read_b128.
//   n-contiguous B: rows of 256 = 32 chunks; logical chunk c of row k sits at chunk c ^ (2 * (k & 7));
//   m-contiguous A of 128 rows: 16 chunks per row; logical chunk c of row k sits at chunk c ^ (4 * (k & 3));
//     these are read with the transposing ds_read_b64_tr_b16, which hands lane i of a 16-lane group the four
//     k-consecutive values of column i of a 4 x 16 block.
//
// The k tiles of all the tiles a workgroup works through form ONE stream through the rings: right after the barrier
// that hands position s to the compute waves, A and B of position s + kSA - 1 are requested, whether or not that belongs
// to the next output tile, so the operand pipeline never drains at a tile boundary.  For the same reason nothing at a tile
// boundary waits for memory: the tile comes out of registers (TileFinder, GroupFinder), gathered row numbers by scalar
// loads.  There is exactly one workgroup barrier per k tile of the stream,
// executed by all the waves.  (An extra barrier at the end of every tile, releasing its last stage before the stores
// so that the loaders request a third k tile during the epilogue, was measured and did not pay.)
//
// With loader waves, a compute wave keeps two register sets of fragments: the LDS reads of k16 step s + 1 are issued
// before the matrix instructions of step s, and the barrier of the next k tile sits in front of the last matrix
// instructions of the current one.
//
// The epilogue needs neither LDS nor barriers: neighbouring lanes exchange one accumulator value through a DPP
// move, so that every lane holds two adjacent columns of one row, and hands them to the policy, which stores them
// (4 bytes of bf16, converted before the exchange, or 8 bytes of fp32 per lane; a half wave writes 64 or 128
// contiguous bytes of each of two rows per instruction).  While the compute waves store, the loaders are already
// up to two k tiles into the next tile.
//
// Workgroups are mapped to tiles XCD-aware: consecutive workgroup ids go round-robin to the 8 XCDs,
// so workgroup id w works for XCD w % 8, and all tiles of one group (block of neurons) are given to
// one XCD, consecutively, so that the group's operand panels are fetched from HBM once and shared in
// that XCD's L2.
#pragma once
#include <type_traits>

#include "common.h"
#include "tile_div.h"

namespace meft {

constexpr int kTN = 256, kTK = 64;
constexpr int kTMTok = 128;            // tile rows of the token-major problems (groups of tokens against a block's rows)
constexpr int kTMNeu = 128;            // tile rows of the router
constexpr int kBSlotElems = kTN * kTK;                         // one B slot: 32 KB
constexpr int kIdRingSlots = 4;                                // k tiles of gathered-row numbers kept per loader
constexpr int kXcd = 8;
// LDS of a launch: the two operand rings and, where the numbers of gathered B rows travel through LDS, 1 KB per
// loading wave
template <class P>
constexpr int operand_lds_bytes() { return (P::kSA * P::kTM + P::kSB * kTN) * kTK * 2; }
template <class P>
constexpr int gemm_lds_bytes() {
  return operand_lds_bytes<P>() + (P::kRowIdsInMemory ? P::kLoaders * kIdRingSlots * 64 * 4 : 0);
}
// threads of a launch: the policy's compute waves plus its loader waves
template <class P>
constexpr int gemm_threads() { return 64 * (P::kCW + P::kLoaders); }

#define MEFT_GPTR(p) ((const __attribute__((address_space(1))) void*)(p))
#define MEFT_LPTR(p) ((__attribute__((address_space(3))) void*)(p))

// Read-only index arrays are read through the constant address space where the index is wave-uniform: that
// makes the load a scalar load, which is counted apart from the vector loads that pace the operand pipeline
// (a vector load would make the compiler wait for every outstanding operand load before using its result).
template <typename T>
__device__ __forceinline__ const __attribute__((address_space(4))) T* as_const(const T* p) {
  return reinterpret_cast<const __attribute__((address_space(4))) T*>(reinterpret_cast<uintptr_t>(p));
}

struct TileCoord {
  int g;       // group (block of neurons); 0 for an ungrouped problem
  int m0, n0;  // first row / column of the tile inside the group's problem
  int Mrows;   // rows of the group's problem
  int Ncols;   // columns of the group's problem
  int nk;      // k tiles
  int slot0;   // first slot of the group in the slot-ordered arrays (token-grouped problems)
  int aux;     // policy-defined
};

// A problem policy P provides:
//   static constexpr int kTM, kSA, kSB;                 tile rows (128) and the slots of the A and B rings (kSA == kSB)
//   static constexpr int kLoaders;                      loader waves, 2 or 4
//   Finder, __device__ Finder finder(int xcd) const;    what a wave of that XCD looks its tiles up with, in registers
//   __device__ bool locate(Finder&, int wg, TileCoord&) const;   false: no tile with id wg, nor with any larger id on
//                                                       the same XCD (ids wg + 8, wg + 16, ...).  Called at every tile
//                                                       boundary of the operand stream: it reads no memory (but for the
//                                                       next part of a group list that is longer than a wave)
//   static constexpr bool kAMC;                         A contiguous along m (rows indexed by k)?
//       false: __device__ const uint16_t* a_row(const TileCoord&, int m, int id) const;    start of row m; id = entry m0 + .. of
//              a_ids where static constexpr bool kAIds is true:
//              __device__ const int32_t* a_ids(const TileCoord&) const;   row numbers of the rows m0 ..  m0 + kTM - 1 (readable
//              and valid also beyond the group);  m < Mrows where it is false
//       true:  __device__ const uint16_t* a_mat() const;                 row 0 of the matrix that holds A,
//              __device__ int a_cols(const TileCoord&) const;            its row length (a multiple of 8), and
//              __device__ int a_krow(const TileCoord&, int k) const;     the number of the row that holds contraction
//              index k (possibly negative; a row of zeros beyond the contraction length)
//   static constexpr bool kBNC;                         B contiguous along n (rows indexed by k)?
//       false: __device__ const uint16_t* b_row(const TileCoord&, int n) const;    start of B row n, n < Ncols;
//              static constexpr bool kBTags: true where B's rows are gathered (buffer loads only):
//              __device__ const int32_t* b_tags(const TileCoord&) const;  for the rows n0 .. n0 + 255 (readable also beyond
//              the block) the number + 1 that b_row takes in n's place, 0 for a row of zeros
//       true:  __device__ const uint16_t* b_row_ptr(int row) const;   start of B row `row`; rows are
//              TileCoord::Ncols elements apart;  and, with static constexpr bool kRowIdsInMemory (false where B
//              is k-contiguous),
//         false: __device__ int b_row_ids(const TileCoord&, int k) const;  number of the B row that holds k (plain
//                arithmetic, no memory access), any valid row for k beyond the contraction length;
//         true:  __device__ const int32_t* b_row_id_src(const TileCoord&, int k0) const;  where the numbers of the B
//                rows of k0 .. k0 + 63 are stored (valid rows also beyond the contraction length: those products are
//                zero); called for k0 = 0, 64, ... below 64 * nk.  The numbers travel like the operands: a
//                4-byte-per-lane global -> LDS load puts the 64 numbers of a k tile into a small ring in LDS one
//                position ahead of the operand request that uses them;
//   __device__ const uint16_t* a_base() const, b_base() const;   lowest address any load of the operand reads;
//   uint32_t a_bytes, b_bytes;  bool buf;               bytes readable from there, and whether both operands are small
//                                                       enough (< 4 GB) for buffer loads (set by set_gemm_extents)
//   __device__ int out_cols(const TileCoord&) const;    columns of the group's output that are stored
//   __device__ int row_tag(const TileCoord&, int m) const;   0: row m of the group's output is not stored (also for
//                m beyond the group's rows); anything else is handed back to row_off.  May read memory: it is asked
//                before the k loop.
//   __device__ size_t row_off(const TileCoord&, int tag, int m) const;   element offset of (row m, column 0) in
//                the output array
//   static constexpr bool kRowsLinear;   true: row_off does not depend on the tag and is linear in m with the step
//                __device__ int out_ld(const TileCoord&) const;   (the kernel then multiplies once per tile)
//   static constexpr bool kOutBf16;   the output is bf16 (the kernel converts, two columns to a word) or fp32
//       false: __device__ void store2(size_t at, int n, float v0, float v1, uint32_t aux) const;   store C[m][n] = v0
//                and C[m][n + 1] = v1 at element offset `at` (= row_off + n; n even, n < round-up of out_cols to 32;
//                the policy checks n and n + 1 against out_cols where that is not a multiple of 32)
//       true:  __device__ void store_pk(size_t at, int n, uint32_t pk, uint32_t aux) const;   the same with
//                pk = bf16(C[m][n]) | bf16(C[m][n + 1]) << 16
//   static constexpr bool kAux;  true: __device__ uint32_t load_aux(const TileCoord&, int m, int n) const;   a word
//                the policy wants next to the two values of (m, n), e.g. a mask; called for every position of the
//                tile, stored or not, so the policy clamps m and n to valid ones
// and for gemm_wide_kernel (kTM 256) instead of the last three
//   __device__ void store16(size_t at, int n, u32x4 v, u32x4 aux) const;   16 bytes of a row at element offset `at` (= row_off + n):
//                eight columns of bf16 (n a multiple of 8) or four of fp32 (a multiple of 4).  The first column of the 64 (fp32: 32)
//                that n is among is below out_cols; the policy checks the rest where out_cols is no multiple of that.  `at` is
//                aligned to four bytes where rows may have an odd length
//   __device__ u32x4 load_aux16(const TileCoord&, int m, int n) const;   (kAux) 16 bytes next to the eight values from (m, n) on, also
//                outside the group and the output, so the policy clamps m and n

// Workgroup barrier of a compute wave: it first waits for its own LDS traffic.  (A loader wave waits for the
// operand loads that have to have landed instead.)
#define MEFT_BARRIER_LDS() asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory")

// P::kCW compute waves (the first waves of the workgroup) and P::kLoaders loader waves (two, or four where the
// loaders' own instruction stream paces the loads: row numbers to look up, an address to form per load).  Measured on gfx950 the
// operand path, not the matrix cores or LDS latency, bounds these
// contractions (a compute unit keeps about a hundred 128-byte read requests in flight on average), and with four
// compute waves a wave that both requests operands and issues MFMAs keeps neither queue full.  The workgroup is persistent: it works through tiles wg, wg + gridDim.x, ...
// (gridDim.x is a multiple of 8, so it stays on one XCD's list).
// kBuf: the operand loads are buffer loads (both operand matrices smaller than 4 GB) instead of global loads
__device__ __forceinline__ uint32_t byte_off(const uint16_t* ptr, const uint16_t* base) {
  return (uint32_t)(reinterpret_cast<uintptr_t>(ptr) - reinterpret_cast<uintptr_t>(base));
}

template <class P, bool kBuf>
__global__ __launch_bounds__(gemm_threads<P>(), 1) void gemm_mfma_kernel(P p, int n_tiles_bound) {
  constexpr int kCW = P::kCW;                       // compute waves: 4 (2 x 2)
  constexpr int kLoaders = P::kLoaders;             // waves that request operands
  constexpr int TM = P::kTM, SA = P::kSA, SB = P::kSB;
  constexpr int WM = TM / (kCW / 2);                // rows of a compute wave
  constexpr int MI = WM / 32;                       // 32-row MFMA tiles per compute wave
  constexpr int kASlotElems = TM * kTK;
  constexpr int kBRing = SA * kASlotElems;          // element offset of the B ring
  static_assert(kLoaders == 2 || kLoaders == 4, "waves that load: 2 or 4");
  static_assert(kCW == 4 && TM == 128, "128 tile rows, 64 to a compute wave");
  static_assert(SA >= 2 && SA <= 3 && SB == SA, "ring depths: 2 or 3, A and B requested for the same positions");
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // locate() answers false only when the workgroup's XCD has no tile with this or any larger id
  typename P::Finder finder = p.finder(blockIdx.x & (kXcd - 1));
  auto next_tile = [&](int wg, TileCoord& t) -> bool { return wg < n_tiles_bound && p.locate(finder, wg, t); };
  const int step = gridDim.x;
  constexpr uint32_t kNowhere = 0xFFFFFFF0u;   // offset outside every buffer: such a load brings zeros and touches no memory

  TileCoord tc;
  if (!next_tile(blockIdx.x, tc)) return;   // the same answer in every wave

  // ---------------------------------------------------------------------- operand requests
  // (state and steps of a loader wave; dead code in the compute waves)
    const int lw = wave - kCW;
    constexpr int LA = TM / 8 / kLoaders;    // A wave-loads (1 KB each) per loader and slot: 8 or 4
    constexpr int LB = kTN / 8 / kLoaders;   // B wave-loads (1 KB each) per loader and slot: 16 or 8
    constexpr int DA = SA - 1;               // positions ahead of the barrier at which they are requested
    constexpr int kAhead = (DA - 1) * (LA + LB);   // loads that may still be in flight at a barrier
    static_assert(kAhead <= 63, "partial vmcnt wait out of range");
    const int lr8 = lane >> 3;
    int* idring = reinterpret_cast<int*>(smem + operand_lds_bytes<P>() / 2) + lw * kIdRingSlots * 64;

    // Cursors over one and the same sequence of (tile, k tile) positions: the operands, and (where they sit in memory) the
    // row numbers of gathered B rows, which run one position ahead.
    struct Cursor {
      int wg, k, n;
      bool ok;
      TileCoord t;
    };
    Cursor cu{(int)blockIdx.x, 0, 0, true, tc}, cd = cu;
    int slot = 0;   // ring slot of the next request
    cd.ok = P::kBNC && P::kRowIdsInMemory;
    //   consume: position handed to the compute waves at the next barrier
    int wg_c = blockIdx.x, nk_c = tc.nk;

    // A, k-contiguous: a wave-load covers 8 rows (m) x 128 bytes; fixed row pointers per tile, advanced by k.
    // A, m-contiguous, 128 rows: a wave-load covers 4 rows (k) x 256 bytes; lane l fetches the 16-byte chunk
    //   (l & 15) ^ (4 * (row & 3)) of its row (the LDS swizzle; row & 3 == (l >> 4) & 3 for every load), so one
    //   column offset per tile serves all the loads.
    // B, k-contiguous: like A, 8 rows (n) x 128 bytes.
    // B, n-contiguous: a wave-load covers two k rows (lanes 0..31 the even one, lanes 32..63 the odd one), 512 bytes
    //   of each; lane l fetches the chunk (l & 31) ^ (2 * (row & 7)); row & 7 only depends on i & 3, so four
    //   column offsets per tile cover all the loads.
    //
    // Every wave-load fills 1 KB of LDS, and the loads of a loader fill consecutive kilobytes.  The instruction's
    // immediate offset is added to the global AND the LDS address (checked on the device), so four consecutive loads
    // share one LDS base (one write of M0 instead of four) with offsets 0, 1, 2, 3 KB, and the global pointers are
    // set up that many bytes lower.
    const uint16_t* pa[P::kAMC ? 4 : LA];   // m-contiguous: row 0 at this lane's column, one per offset 0..3 KB
    const uint16_t* pb[P::kBNC ? 4 : LB];
    // Buffer loads (kBuf): the same addresses as 32-bit byte offsets from the operand's lowest address, without the
    // kilobyte shifts (every load writes M0, a scalar instruction).  Whatever is the same in all lanes goes into the
    // instruction's scalar offset: the k offset of k-contiguous operands, the row offset of consecutive B rows.
    [[maybe_unused]] uint32_t oa[P::kAMC ? 4 : LA], ob[P::kBNC ? 4 : LB];
    const int half = lane >> 5;
    // Rows beyond the group are not loaded (buffer loads), or any valid row is.  Gathered row numbers come by scalar loads,
    // eight per wave-load, of which each lane picks its row's: a vector load here would wait for every operand request on
    // its way.
    [[maybe_unused]] auto id_of_row = [&](const int32_t* ids8) -> int {   // of this lane's row among a wave-load's eight
      const auto* ids = as_const(ids8);
      int s[8];
#pragma unroll
      for (int z = 0; z < 8; ++z) s[z] = ids[z];
      const int s01 = (lr8 & 1) ? s[1] : s[0], s23 = (lr8 & 1) ? s[3] : s[2], s45 = (lr8 & 1) ? s[5] : s[4],
                s67 = (lr8 & 1) ? s[7] : s[6];
      const int s03 = (lr8 & 2) ? s23 : s01, s47 = (lr8 & 2) ? s67 : s45;
      return (lr8 & 4) ? s47 : s03;
    };
    [[maybe_unused]] auto a_row_start = [&](const TileCoord& t, int i) -> const uint16_t* {
      if constexpr (P::kAMC) {
        return nullptr;
      } else {
      const int row = (lw * LA + i) * 8 + lr8;
      int id = 0, m = t.m0 + row;
      if constexpr (P::kAIds) {
        id = id_of_row(p.a_ids(t) + (lw * LA + i) * 8);
      } else {
        m = m < t.Mrows ? m : t.Mrows - 1;
      }
      return p.a_row(t, m, id) + (((lane & 7) ^ ((row >> 1) & 7)) << 3);
      }
    };
    auto setup_a = [&]() {
      const TileCoord& t = cu.t;
      if constexpr (kBuf) {
        if constexpr (P::kAMC) {
          const int chunk = (lane & 15) ^ (4 * ((lane >> 4) & 3));
          const int col = t.m0 + chunk * 8, last = p.a_cols(t) - 8;
          const uint32_t o = byte_off(p.a_mat() + (col > last ? last : col), p.a_base());
#pragma unroll
          for (int q = 0; q < 4; ++q) oa[q] = o;
        } else {
#pragma unroll
          for (int i = 0; i < LA; ++i) {
            const uint32_t o = byte_off(a_row_start(t, i), p.a_base());
            oa[i] = t.m0 + (lw * LA + i) * 8 + lr8 < t.Mrows ? o : kNowhere;
          }
        }
      } else {
        if constexpr (P::kAMC) {
          const int chunk = (lane & 15) ^ (4 * ((lane >> 4) & 3));
          const int col = t.m0 + chunk * 8, last = p.a_cols(t) - 8;
          const int acol = col > last ? last : col;                       // clamp (rows beyond Mrows are never stored)
#pragma unroll
          for (int q = 0; q < 4; ++q) pa[q] = p.a_mat() + (acol - q * 512);
        } else {
#pragma unroll
          for (int i = 0; i < LA; ++i) pa[i] = a_row_start(t, i) - (i & 3) * 512;
        }
      }
    };
    auto setup_b = [&]() {
      const TileCoord& t = cu.t;
      if constexpr (kBuf) {
        if constexpr (P::kBNC) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int chunk = (lane & 31) ^ (2 * ((2 * q + half) & 7));
            int col = t.n0 + chunk * 8;
            col = col > t.Ncols - 8 ? t.Ncols - 8 : col;
            ob[q] = byte_off(p.b_row_ptr(0) + col, p.b_base());
          }
        } else {
#pragma unroll
          for (int i = 0; i < LB; ++i) {
            const int row = (lw * LB + i) * 8 + lr8, n = min(t.n0 + row, t.Ncols - 1);
            const int swz = ((lane & 7) ^ ((row >> 1) & 7)) << 3;
            // (no branch that differs per lane: see TileFinder::load)
            int from = n, there = t.n0 + row < t.Ncols ? 1 : 0;
            if constexpr (P::kBTags) {
              const int tag = id_of_row(p.b_tags(t) + (lw * LB + i) * 8);
              there &= tag > 0 ? 1 : 0;
              from = max(tag, 1) - 1;
            }
            const uint32_t o = byte_off(p.b_row(t, from) + swz, p.b_base());
            ob[i] = there ? o : kNowhere;
          }
        }
      } else {
        if constexpr (P::kBNC) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int chunk = (lane & 31) ^ (2 * ((2 * q + half) & 7));
            int col = t.n0 + chunk * 8;
            col = col > t.Ncols - 8 ? t.Ncols - 8 : col;              // clamp (columns beyond Ncols are never stored)
            pb[q] = p.b_row_ptr(0) + col - q * 512;
          }
        } else {
#pragma unroll
          for (int i = 0; i < LB; ++i) {
            const int row = (lw * LB + i) * 8 + lr8, n = min(t.n0 + row, t.Ncols - 1);
            pb[i] = p.b_row(t, n) + (((lane & 7) ^ ((row >> 1) & 7)) << 3) - (i & 3) * 512;
          }
        }
      }
    };
    // Where every operand matrix is smaller than 4 GB the loads are buffer loads (a wave-uniform resource descriptor,
    // a 32-bit offset per lane and a scalar offset instead of a 64-bit address per lane): the vector-memory path
    // takes them faster (score GEMM 0.331 -> 0.314 ms), and a load of the k-contiguous problems then costs the
    // loader a write of M0 and nothing else.
    __amdgpu_buffer_rsrc_t rsrc_a = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p.a_base()), 0, (int)p.a_bytes, 0x00020000);
    __amdgpu_buffer_rsrc_t rsrc_b = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p.b_base()), 0, (int)p.b_bytes, 0x00020000);
    // load number i of a loader into the 1 KB slot i of its part of an operand region (see above)
    // (the offset has to be a literal: the switch folds away once the loop over i is unrolled)
#define MEFT_LOAD_1K(src, region, i)                                                    \
  do {                                                                                  \
    const auto* g_ = MEFT_GPTR(src);                                                    \
    auto* l_ = MEFT_LPTR((region) + ((i) & ~3) * 512);                                  \
    switch ((i) & 3) {                                                                  \
      case 0: __builtin_amdgcn_global_load_lds(g_, l_, 16, 0, 0); break;                \
      case 1: __builtin_amdgcn_global_load_lds(g_, l_, 16, 1024, 0); break;             \
      case 2: __builtin_amdgcn_global_load_lds(g_, l_, 16, 2048, 0); break;             \
      default: __builtin_amdgcn_global_load_lds(g_, l_, 16, 3072, 0); break;            \
    }                                                                                   \
  } while (0)
    // buffer load number i: lane offset `voff`, wave-uniform offset `soff` (bytes).  The casts are needed: handed an
    // unsigned offset, this toolchain's host pass drops the kernel's launch stub without any diagnostic and the
    // library then fails to load with an undefined symbol.
#define MEFT_LOAD_1K_BUF(rsrc, voff, soff, region, i) \
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, MEFT_LPTR((region) + (i) * 512), 16, (int)(voff), (int)(soff), 0, 0)

    auto request_ids = [&]() {
      if constexpr (P::kBNC && P::kRowIdsInMemory) {
        if (!cd.ok) return;
        __builtin_amdgcn_global_load_lds(MEFT_GPTR(p.b_row_id_src(cd.t, cd.k * kTK) + lane),
                                         MEFT_LPTR(idring + (cd.n & (kIdRingSlots - 1)) * 64), 4, 0, 0);
        ++cd.n;
        if (++cd.k == cd.t.nk) { cd.wg += step; cd.k = 0; cd.ok = next_tile(cd.wg, cd.t); }
      }
    };
    // one k tile of A into the next slot of the A ring
    auto request_a = [&]() {
      const TileCoord& t = cu.t;
      uint16_t* my_a = smem + slot * kASlotElems + lw * LA * 512;   // 512 elements = 1 KB per load
      [[maybe_unused]] int a_row_bytes = 0;
      if constexpr (P::kAMC) a_row_bytes = p.a_cols(t) * 2;
      if constexpr (kBuf) {
        const int k_bytes = cu.k * kTK * 2;
#pragma unroll
        for (int i = 0; i < LA; ++i) {
          if constexpr (P::kAMC) {
            const int row = p.a_krow(t, cu.k * kTK + 4 * (lw * LA + i) + (lane >> 4));
            MEFT_LOAD_1K_BUF(rsrc_a, oa[i & 3] + (uint32_t)row * (uint32_t)a_row_bytes, 0, my_a, i);
          } else {
            MEFT_LOAD_1K_BUF(rsrc_a, oa[i], k_bytes, my_a, i);
          }
        }
      } else {
#pragma unroll
        for (int i = 0; i < LA; ++i) {
          if constexpr (P::kAMC) {
            const int row = p.a_krow(t, cu.k * kTK + 4 * (lw * LA + i) + (lane >> 4));
            MEFT_LOAD_1K(reinterpret_cast<const char*>(pa[i & 3]) + (int64_t)row * a_row_bytes, my_a, i);
          } else {
            MEFT_LOAD_1K(pa[i] + cu.k * kTK, my_a, i);
          }
        }
      }
    };
    // one k tile of B into the next slot of the B ring
    auto request_b = [&]() {
      const TileCoord& t = cu.t;
      // n-contiguous B: ids[i] = number of the B row this lane fetches in its i-th load,
      // k = 64 * cu.k + 2 * (lw * LB + i) + half
      int ids[LB];
      if constexpr (P::kBNC && P::kRowIdsInMemory) {
        // out of the ring; one asm block with its own wait (through plain loads the compiler would first drain every
        // outstanding operand load)
        const uint32_t a = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)(
            idring + (cu.n & (kIdRingSlots - 1)) * 64 + 2 * lw * LB + half);
        if constexpr (LB == 16) {
        asm volatile(
            "ds_read_b32 %0, %16\n\tds_read_b32 %1, %16 offset:8\n\tds_read_b32 %2, %16 offset:16\n\t"
            "ds_read_b32 %3, %16 offset:24\n\tds_read_b32 %4, %16 offset:32\n\tds_read_b32 %5, %16 offset:40\n\t"
            "ds_read_b32 %6, %16 offset:48\n\tds_read_b32 %7, %16 offset:56\n\tds_read_b32 %8, %16 offset:64\n\t"
            "ds_read_b32 %9, %16 offset:72\n\tds_read_b32 %10, %16 offset:80\n\tds_read_b32 %11, %16 offset:88\n\t"
            "ds_read_b32 %12, %16 offset:96\n\tds_read_b32 %13, %16 offset:104\n\tds_read_b32 %14, %16 offset:112\n\t"
            "ds_read_b32 %15, %16 offset:120\n\ts_waitcnt lgkmcnt(0)"
            : "=&v"(ids[0]), "=&v"(ids[1]), "=&v"(ids[2]), "=&v"(ids[3]), "=&v"(ids[4]), "=&v"(ids[5]), "=&v"(ids[6]),
              "=&v"(ids[7]), "=&v"(ids[8]), "=&v"(ids[9]), "=&v"(ids[10]), "=&v"(ids[11]), "=&v"(ids[12]),
              "=&v"(ids[13]), "=&v"(ids[14]), "=&v"(ids[15])
            : "v"(a)
            : "memory");
        } else {
        static_assert(LB == 16 || LB == 8, "row-number reads are written out for 16 and 8 loads");
        asm volatile(
            "ds_read_b32 %0, %8\n\tds_read_b32 %1, %8 offset:8\n\tds_read_b32 %2, %8 offset:16\n\t"
            "ds_read_b32 %3, %8 offset:24\n\tds_read_b32 %4, %8 offset:32\n\tds_read_b32 %5, %8 offset:40\n\t"
            "ds_read_b32 %6, %8 offset:48\n\tds_read_b32 %7, %8 offset:56\n\ts_waitcnt lgkmcnt(0)"
            : "=&v"(ids[0]), "=&v"(ids[1]), "=&v"(ids[2]), "=&v"(ids[3]), "=&v"(ids[4]), "=&v"(ids[5]), "=&v"(ids[6]),
              "=&v"(ids[7])
            : "v"(a)
            : "memory");
        }
      } else if constexpr (P::kBNC) {
#pragma unroll
        for (int i = 0; i < LB; ++i) ids[i] = p.b_row_ids(t, cu.k * kTK + 2 * (lw * LB + i) + half);
      }
      uint16_t* my_b = smem + kBRing + slot * kBSlotElems + lw * LB * 512;
      if constexpr (kBuf) {
        const int k_bytes = cu.k * kTK * 2;
        if constexpr (P::kBNC) {
          const uint32_t row_bytes = (uint32_t)t.Ncols * 2u;
          bool linear = false;
          if constexpr (!P::kRowIdsInMemory) {
            linear = p.b_rows_linear(t, cu.k * kTK);
            if (linear) {
              // 64 consecutive rows: this lane's row is first + 2 * (lw * LB + i) + half
              const uint32_t first = (uint32_t)p.b_row_ids(t, cu.k * kTK) * row_bytes, hoff = half * row_bytes;
#pragma unroll
              for (int i = 0; i < LB; ++i)
                MEFT_LOAD_1K_BUF(rsrc_b, ob[i & 3] + hoff, (int)(first + 2u * (lw * LB + i) * row_bytes), my_b, i);
            }
          }
          if (!linear) {
#pragma unroll
            for (int i = 0; i < LB; ++i)
              MEFT_LOAD_1K_BUF(rsrc_b, ob[i & 3] + (uint32_t)ids[i] * row_bytes, 0, my_b, i);
          }
        } else {
#pragma unroll
          for (int i = 0; i < LB; ++i) MEFT_LOAD_1K_BUF(rsrc_b, ob[i], k_bytes, my_b, i);
        }
      } else {
        if constexpr (P::kBNC) {
          const uint32_t row_bytes = (uint32_t)t.Ncols * 2u;
#pragma unroll
          for (int i = 0; i < LB; ++i)
            MEFT_LOAD_1K(reinterpret_cast<const char*>(pb[i & 3]) + (uint64_t)(uint32_t)ids[i] * row_bytes, my_b, i);
        } else {
#pragma unroll
          for (int i = 0; i < LB; ++i) MEFT_LOAD_1K(pb[i] + cu.k * kTK, my_b, i);
        }
      }
    };
    // one k tile of each operand; false: the stream has ended, nothing was requested
    auto request_operands = [&]() -> bool {
      if (!cu.ok) return false;
      request_a();
      request_b();
      ++cu.n;
      slot = slot + 1 == SA ? 0 : slot + 1;
      if (++cu.k == cu.t.nk) {
        cu.wg += step; cu.k = 0; cu.ok = next_tile(cu.wg, cu.t);
        if (cu.ok) { setup_a(); setup_b(); }
      }
      return true;
    };
    // the requests that follow a barrier
    auto request_batch = [&]() -> bool {
      request_ids();
      return request_operands();
    };

  if (wave >= kCW) {
    setup_a();
    setup_b();
    if constexpr (P::kBNC && P::kRowIdsInMemory) {
#pragma unroll
      for (int s = 0; s < DA + 1; ++s) request_ids();
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    bool full = true;   // before the first barrier: the positions the lead reaches
#pragma unroll
    for (int s = 0; s < DA; ++s) full = request_operands() && full;

    // ------------------------------------------------------------------ loader waves
    for (;;) {
      for (int kt = 0; kt < nk_c; ++kt) {
        // The position handed over now has landed once at most the kAhead most recent loads are outstanding (the
        // counter retires in issue order), provided the last batch of requests was complete; near the end of the
        // stream everything is awaited.
        if (full) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(kAhead) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
        // every compute wave is past the previous position: its slots are free
        full = request_batch();
      }
      wg_c += step;
      TileCoord t;
      if (!next_tile(wg_c, t)) return;
      nk_c = t.nk;
    }
  }

  // -------------------------------------------------------------------- compute waves
  const int wm = (wave >> 1) * WM, wn = (wave & 1) * 128;
  const int fr = lane & 31, fc = lane >> 5;
  // k-contiguous operands: element offsets of this lane's fragment rows inside a slot, and their swizzle keys
  int offA[MI], keyA[MI], offB[4], keyB[4];
#pragma unroll
  for (int i = 0; i < MI; ++i) { const int r = wm + i * 32 + fr; offA[i] = r * kTK; keyA[i] = (r >> 1) & 7; }
#pragma unroll
  for (int j = 0; j < 4; ++j) { const int r = wn + j * 32 + fr; offB[j] = r * kTK; keyB[j] = (r >> 1) & 7; }
  // m- / n-contiguous operands: LDS byte offsets (inside a slot) of this lane's transposing reads.  Lane s of a
  // 16-lane group points at row (k base + s/4), columns 4*(s%4)..+3 of a 4 x 16 block and receives column s of that
  // block, four consecutive k.  Low half: k = 8*(lane/32) + 0..3, high half +4.
  uint32_t tra_lo[2], tra_hi[2], tr_lo[4], tr_hi[4];
  {
    const int gq = lane >> 4, s = lane & 15;
    const int k_lo = 8 * (gq >> 1) + (s >> 2), k_hi = k_lo + 4;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int m = wm + i * 32 + 16 * (gq & 1) + 4 * (s & 3);
      const int x_lo = 4 * (k_lo & 3), x_hi = 4 * (k_hi & 3);
      tra_lo[i] = (uint32_t)(k_lo * TM + (((m >> 3) ^ x_lo) << 3) + (m & 7)) * 2u;
      tra_hi[i] = (uint32_t)(k_hi * TM + (((m >> 3) ^ x_hi) << 3) + (m & 7)) * 2u;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n = wn + j * 32 + 16 * (gq & 1) + 4 * (s & 3);
      tr_lo[j] = (uint32_t)(k_lo * kTN + (((n >> 3) ^ (2 * (k_lo & 7))) << 3) + (n & 7)) * 2u;
      tr_hi[j] = (uint32_t)(k_hi * kTN + (((n >> 3) ^ (2 * (k_hi & 7))) << 3) + (n & 7)) * 2u;
    }
  }

  int wg = blockIdx.x;
  int slot_a = 0, slot_b = 0;   // run on across tiles, like the loaders' slots
  for (;;) {
    // lane l: the tag of row wm + l of this tile.  Asked before the k loop, so that a policy's memory read has long
    // returned when the answer is needed.
    const int my_tag = p.row_tag(tc, tc.m0 + wm + lane);

    f32x16 acc[MI][4];
    const int nk = tc.nk;
    // The fragments of one k16 step.  Two sets alternate: the LDS reads of step s + 1 are issued before the matrix
    // instructions of step s, so that their latency passes under those 8 instructions instead of in front of
    // the next ones.  (Left to itself the compiler reads each step's fragments into the same registers right before
    // their use, and the matrix pipe idles for an LDS round trip four times per k tile.)
    struct Frags { bf16x8 a[MI], b[4]; };
    Frags f0, f1;
    constexpr uint32_t kStepA = 16 * TM * 2;   // bytes of 16 k rows of an m-contiguous A slot
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    // transposing read of this lane's 8 values of one operand fragment: low and high k half, 8 bytes each
    auto tr_pair = [&](const uint16_t* slot, uint32_t lo_off, uint32_t hi_off) -> bf16x8 {
      const auto* base = (const __attribute__((address_space(3))) char*)(slot);
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(base + lo_off));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(base + hi_off));
      return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    // issue the LDS reads of k16 step KS of the current slots
    auto load_frags = [&](auto ks_tag, Frags& f) {
      constexpr int ks = decltype(ks_tag)::value;
      const uint16_t* sta = smem + slot_a * kASlotElems;
      const uint16_t* stb = smem + kBRing + slot_b * kBSlotElems;
      const int c = ks * 2 + fc;   // k-contiguous operands: this lane's 16-byte chunk of the k16 step
      // k16 step ks starts 16 rows further (B: 8192 bytes, m-contiguous A: 4096 or 8192 bytes); that changes neither
      // (k & 7) nor (k & 3), so the swizzles hold
      if constexpr (!P::kAMC) {
#pragma unroll
        for (int i = 0; i < MI; ++i) f.a[i] = *reinterpret_cast<const bf16x8*>(&sta[offA[i] + ((c ^ keyA[i]) << 3)]);
      } else {
        static_assert(!P::kAMC || P::kBNC, "an m-contiguous A comes with an n-contiguous B");
#pragma unroll
        for (int i = 0; i < 2; ++i) f.a[i] = tr_pair(sta, tra_lo[i] + ks * kStepA, tra_hi[i] + ks * kStepA);
      }
      if constexpr (!P::kBNC) {
#pragma unroll
        for (int j = 0; j < 4; ++j) f.b[j] = *reinterpret_cast<const bf16x8*>(&stb[offB[j] + ((c ^ keyB[j]) << 3)]);
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) f.b[j] = tr_pair(stb, tr_lo[j] + ks * 8192u, tr_hi[j] + ks * 8192u);
      }
    };
    // kZero: the step starts from zero instead of from acc (the matrix instruction takes the constant as its addend,
    // so the accumulators are never cleared by hand)
    auto mma = [&](auto zero_tag, const Frags& f) {
      constexpr bool kZero = decltype(zero_tag)::value;
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if constexpr (kZero) {
            const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[i], f.b[j], zero, 0, 0, 0);
          } else {
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[i], f.b[j], acc[i][j], 0, 0, 0);
          }
        }
    };
    // nothing moves across: the order of reads and matrix instructions below is the schedule
#define MEFT_FENCE() __builtin_amdgcn_sched_barrier(0)
    // Steps 0..2 of a k tile whose first fragments (f0) are on their way; its step 3 (f1) is left to the caller.
    auto k_steps = [&](auto first_tag) {
      load_frags(std::integral_constant<int, 1>{}, f1);
      MEFT_FENCE();
      mma(first_tag, f0);
      MEFT_FENCE();
      load_frags(std::integral_constant<int, 2>{}, f0);
      MEFT_FENCE();
      mma(std::false_type{}, f1);
      MEFT_FENCE();
      load_frags(std::integral_constant<int, 3>{}, f1);
      MEFT_FENCE();
      mma(std::false_type{}, f0);
      MEFT_FENCE();
      slot_a = slot_a + 1 == SA ? 0 : slot_a + 1;
      slot_b = slot_b + 1 == SB ? 0 : slot_b + 1;
    };
    MEFT_BARRIER_LDS();   // the loaders have seen the tile's first k tile land
    load_frags(std::integral_constant<int, 0>{}, f0);
    MEFT_FENCE();
    k_steps(std::true_type{});
    for (int kt = 1; kt < nk; ++kt) {
      // The barrier for k tile kt sits in front of the last matrix instructions of k tile kt - 1: every LDS read of
      // that position has returned (the barrier macro waits for them), so the loaders may have its slots, and the
      // first reads of the new position pass under those instructions.
      MEFT_BARRIER_LDS();
      load_frags(std::integral_constant<int, 0>{}, f0);
      MEFT_FENCE();
      mma(std::false_type{}, f1);
      MEFT_FENCE();
      k_steps(std::false_type{});
    }
    mma(std::false_type{}, f1);
#undef MEFT_FENCE

    // ---- epilogue, out of the registers.  acc[i][j][r] is C[m][n] with m = wm + i*32 + (r/4)*8 + (lane/32)*4 + r%4
    // and n = wn + j*32 + lane%32.  For a register pair (r, r+1), r even, an even lane (column c) keeps its value of
    // row m and takes its right neighbour's value of that row; the odd lane (column c+1) keeps its value of row m+1
    // and takes its left neighbour's (DPP quad_perm [1,0,3,2] swaps neighbours).  Both then hold columns (c, c+1) of
    // one row.  Per 32 rows of the accumulators (i), four register pairs at a time, the rows' tags and whatever the
    // policy reads per element (load_aux: unconditional loads, all in flight together) are fetched first, then the
    // values are exchanged and stored.
    {
      const bool odd = (lane & 1) != 0;
      const int nj = (p.out_cols(tc) - (tc.n0 + wn) + 31) / 32;   // 32-column fragments of this wave with stored columns
      const int ncol = tc.n0 + wn + (fr & ~1);
      // row of this lane inside the wave's rows = lane_row + a constant of the register pair
      const int lane_row = fc * 4 + (lane & 1);
      [[maybe_unused]] size_t lane_at = 0;
      [[maybe_unused]] int ld = 0;
      if constexpr (P::kRowsLinear) {
        ld = p.out_ld(tc);
        lane_at = p.row_off(tc, 1, tc.m0 + wm + lane_row) + ncol;   // one multiplication per tile
      }
      [[maybe_unused]] const unsigned long long ok_mask = __ballot(my_tag != 0);
      auto epilogue = [&](auto full_tag) {
        constexpr bool kFull = decltype(full_tag)::value;   // all four fragments of the wave lie inside the output
#pragma unroll
        for (int i = 0; i < MI; ++i) {
#pragma unroll
          for (int qh = 0; qh < 2; ++qh) {
            int tag[4];
            uint32_t aux[4][4];
#pragma unroll
            for (int qq = 0; qq < 4; ++qq) {
              const int r = 2 * (qh * 4 + qq);
              const int rl = i * 32 + (r >> 2) * 8 + (r & 3) + lane_row;
              // the row's tag: a bit of the wave's ballot where it only says "stored or not" (no trip through the LDS
              // pipeline, which the loaders keep busy), a lane permute where it carries a number
              if constexpr (P::kRowsLinear) {
                tag[qq] = (int)((ok_mask >> rl) & 1ull);
              } else {
                tag[qq] = __builtin_amdgcn_ds_bpermute(rl << 2, my_tag);
              }
              if constexpr (P::kAux) {
#pragma unroll
                for (int j = 0; j < 4; ++j) aux[qq][j] = p.load_aux(tc, tc.m0 + wm + rl, ncol + 32 * j);
              } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) aux[qq][j] = 0u;
              }
            }
#pragma unroll
            for (int qq = 0; qq < 4; ++qq) {
              const int r = 2 * (qh * 4 + qq);
              const int rc = i * 32 + (r >> 2) * 8 + (r & 3);   // the register pair's constant part of the row
              [[maybe_unused]] uint32_t pk[4];
              [[maybe_unused]] float lo[4], hi[4];
              if constexpr (P::kOutBf16) {
                // bf16 output: both rows' values of this lane's column are packed first, (row m | row m+1 << 16); one
                // neighbour swap of the packed word and one byte permute give (column c | column c+1 << 16) of the
                // lane's row (even lanes: row m from the low halves, odd lanes: row m+1 from the high halves)
                const uint32_t sel = odd ? 0x03020706u : 0x05040100u;   // bytes 0-3: own word, 4-7: the neighbour's
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                  const uint32_t own = pack_bf16x2(acc[i][j][r], acc[i][j][r + 1]);
                  const uint32_t nb = (uint32_t)__builtin_amdgcn_update_dpp((int)own, (int)own, 0xB1, 0xF, 0xF, true);
                  pk[j] = __builtin_amdgcn_perm(nb, own, sel);
                }
              } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                  const float a = acc[i][j][r], b = acc[i][j][r + 1];   // plain copies: the values go to the builtin as floats
                  const float an = __builtin_amdgcn_update_dpp(a, a, 0xB1, 0xF, 0xF, true);   // the neighbour's a
                  const float bn = __builtin_amdgcn_update_dpp(b, b, 0xB1, 0xF, 0xF, true);   // the neighbour's b
                  lo[j] = odd ? bn : a;
                  hi[j] = odd ? b : an;
                }
              }
              if (tag[qq] != 0) {
                size_t at;
                if constexpr (P::kRowsLinear) at = lane_at + (size_t)(rc * ld);   // rc * ld: scalar arithmetic
                else at = p.row_off(tc, tag[qq], tc.m0 + wm + rc + lane_row) + ncol;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                  if (kFull || j < nj) {
                    if constexpr (P::kOutBf16) p.store_pk(at + 32 * j, ncol + 32 * j, pk[j], aux[qq][j]);
                    else p.store2(at + 32 * j, ncol + 32 * j, lo[j], hi[j], aux[qq][j]);
                  }
                }
              }
            }
          }
        }
      };
      if (nj >= 4) epilogue(std::true_type{});
      else epilogue(std::false_type{});
    }
    wg += step;
    if (!next_tile(wg, tc)) break;
  }
}

// ---- tile schedule shared by the grouped problems ----------------------------------------------
// Every non-empty group (block of neurons with its tokens) is given to one XCD; XCD x works through its list
// in order.  grp[x][i] = (group, first slot, rows, number of 128-row m tiles of the groups before it in this list); an
// end entry (-1, ., ., total m tiles) closes the list.  tiles[x][i] counts the m tiles in 64 and in 128 rows.  Inside a group the m tiles vary fastest, so that the tiles that share a
// B panel (one n tile of the group's block) run at the same time and the panel is read from HBM once.
//
// Groups differ in size (the router does not balance them), so they are dealt out longest first, each to the
// XCD with the least work so far (ties to the lower XCD); the work of a group is counted in 64-row units plus
// a constant for the per-tile overhead, which balances both the token-major tile counts and the contraction
// lengths of the neuron-major problems.  Which XCD computes a group has no influence on any result.
//
// Groups of at most `small_rows` tokens come last in every list (the deal runs from the longest group down), and a
// second set of list lengths counts only the larger groups in front of them: a problem that leaves the small groups
// to the per-pair kernels (small_groups.h) walks that prefix of the same lists.
struct TokenSched {
  const int4* grp;       // [kXcd][cap]: group, its first slot, its rows, 128-row m tiles of the groups before it
  const int2* tiles;     // [kXcd][cap]: 64-row and 128-row m tiles of the groups before it
  const int* len;        // [kXcd] number of groups in the list; [kXcd]: 1 = every list holds every group (split);
                         // [kXcd + 1 + x]: groups of more than small_rows tokens in XCD x's list (a prefix of it)
  int cap;               // entries per XCD (n_groups + 1)
  int max_tiles;         // upper bound of m tiles of one XCD (for the tile-id bound of a launch)
};
constexpr int kSchedLenInts = 2 * kXcd + 1;

constexpr int kSchedSortMax = 1024;   // up to this many groups are dealt out longest first; more: round-robin

__device__ __forceinline__ void sched_entry(int4* __restrict__ grp, int2* __restrict__ tiles, size_t at, int g, int slot0,
                                            int rows, int t64, int t128) {
  grp[at] = make_int4(g, slot0, rows, t128);
  tiles[at] = make_int2(t64, t128);
}

// Executed by one whole workgroup of 1024 threads; rows, slot0 = number of tokens and first slot of group threadIdx.x
// (0 rows beyond n_groups).  n_groups <= kSchedSortMax.
// One workgroup, once: what it costs is chains of instructions.  The ranks are counted by all threads, the deal proper is the
// only serial part (scalar registers; a wave-wide arg-min per group took 110 ns each), and the lists are written by a wave per
// XCD.  The workgroup that does this and the tables before it:
// 15.5 -> 10 us with 64 groups, 24 -> 17 with 168 of 256.
__device__ __forceinline__ void build_sched_body(int rows, int slot0, int n_groups, int cap, int4* __restrict__ grp,
                                                 int2* __restrict__ tiles, int* __restrict__ len, int small_rows) {
  __shared__ int s_rows[kSchedSortMax];
  __shared__ int s_slot[kSchedSortMax];
  __shared__ int s_rank[kSchedSortMax];
  __shared__ int s_order[kSchedSortMax];
  __shared__ int s_sorted[kSchedSortMax];
  const int tid = threadIdx.x, lane = tid & 63;
  __syncthreads();   // the arrays may still be read from an earlier use
  if (tid < n_groups) { s_rows[tid] = rows; s_slot[tid] = slot0; s_rank[tid] = 0; }
  const int n_full = __syncthreads_count(rows > 0);   // non-empty groups; also orders the writes above
  {
    // position in the order (rows descending, group id ascending): a permutation.  Thread (part, g) counts the groups part,
    // part + parts, ... before group g.
    const int lg = n_groups > 1 ? 32 - __clz(n_groups - 1) : 0, g = tid & ((1 << lg) - 1), parts = 1024 >> lg;
    if (g < n_groups) {
      const int mine = s_rows[g];
      int before = 0;
#pragma unroll 4
      for (int o = tid >> lg; o < n_groups; o += parts) before += s_rows[o] > mine - (o < g ? 1 : 0) ? 1 : 0;
      if (before) atomicAdd(&s_rank[g], before);
    }
  }
  __syncthreads();
  if (tid < n_groups) {
    s_order[s_rank[tid]] = tid;
    s_sorted[s_rank[tid]] = rows;
  }
  __syncthreads();
  // Fewer non-empty groups than XCDs: a deal of whole groups would leave XCDs idle.  Then every list holds every
  // group, len[kXcd] says so, and XCD x takes the tiles x, x + 8, ... of each group (TileFinder, GroupFinder) or a consecutive
  // part of all of them (WideFinder).
  const bool split = n_full < kXcd;
  if (tid == 0) len[kXcd] = split ? 1 : 0;
  if (split) {
    if (tid < kXcd) {
      int t64 = 0, t128 = 0, n_big = 0;
      for (int i = 0; i < n_full; ++i) {
        const int g = s_order[i], r = s_sorted[i];
        sched_entry(grp, tiles, (size_t)tid * cap + i, g, s_slot[g], r, t64, t128);
        n_big += r > small_rows ? 1 : 0;
        t64 += (r + 63) >> 6;
        t128 += (r + 127) >> 7;
      }
      sched_entry(grp, tiles, (size_t)tid * cap + n_full, -1, 0, 0, t64, t128);
      len[tid] = n_full;
      len[kXcd + 1 + tid] = n_big;
    }
    return;
  }
  int* s_xcd = s_rank;   // XCD of the i-th group of the order
  if (tid < 64) {
    // The groups of more than 64 rows one after another: each to the XCD with the least load (in units of 64 rows plus a
    // constant per group; ties to the lower XCD).  key[0] < key[1] < ... are the loads * 8 + XCD; the first one grows by the
    // group's weight and is put back in its place.
    int n_deal = 0;
    for (int i0 = 0; i0 < n_full; i0 += 64) n_deal += __popcll(__ballot(i0 + lane < n_full && s_sorted[min(i0 + lane, n_full - 1)] > 64));
    int key[kXcd];
#pragma unroll
    for (int x = 0; x < kXcd; ++x) key[x] = x;
    for (int i0 = 0; i0 < n_deal; i0 += 64) {
      const int m = min(64, n_deal - i0), r = s_sorted[min(i0 + lane, n_deal - 1)];
      const int inc = (((r + 63) >> 6) + 2) << 3;
      int xcd = 0;
      for (int i = 0; i < m; ++i) {
        int k = key[0];
        xcd = lane == i ? k & (kXcd - 1) : xcd;
        k += __builtin_amdgcn_readlane(inc, i);
#pragma unroll
        for (int x = 1; x < kXcd; ++x) {
          key[x - 1] = min(k, key[x]);
          k = max(k, key[x]);
        }
        key[kXcd - 1] = k;
      }
      if (lane < m) s_xcd[i0 + lane] = xcd;
    }
    // The groups of at most 64 rows all weigh the same (3), so the same deal has a closed form: XCD x takes its j-th one
    // (from 0) when the least load is load[x] + 3 j, and that is group number
    // sum over y of #{j' : (load[y] + 3 j', y) < (load[x] + 3 j, x)} of the rest.
    const int n_eq = n_full - n_deal, x8 = lane & (kXcd - 1);
    int my_load = 0;
#pragma unroll
    for (int y = 0; y < kXcd; ++y) my_load = (key[y] & (kXcd - 1)) == x8 ? key[y] >> 3 : my_load;
    for (int j0 = 0; j0 < n_eq; j0 += 8) {
      const int k = my_load + 3 * (j0 + (lane >> 3));
      int rank = 0;
#pragma unroll
      for (int y = 0; y < kXcd; ++y) {
        const int v = k - (key[y] >> 3) + ((key[y] & (kXcd - 1)) < x8 ? 1 : 0);
        rank += v > 0 ? (v + 2) / 3 : 0;
      }
      if (!__ballot(rank < n_eq)) break;
      if (rank < n_eq) s_xcd[n_deal + rank] = x8;
    }
  }
  __syncthreads();
  const int x = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (x >= kXcd) return;
  int n = 0, t64 = 0, t128 = 0, n_big = 0;
  for (int i0 = 0; i0 < n_full; i0 += 64) {
    const int at = min(i0 + lane, n_full - 1), r = s_sorted[at], g = s_order[at];
    const bool mine = i0 + lane < n_full && s_xcd[at] == x;
    const unsigned long long mask = __ballot(mine);
    const int u = (r + 63) >> 6, t = (r + 127) >> 7;
    const int iu = wave_incl_scan(mine ? u : 0), it = wave_incl_scan(mine ? t : 0);
    if (mine)
      sched_entry(grp, tiles, (size_t)x * cap + n + __popcll(mask & ((1ull << lane) - 1ull)), g, s_slot[g], r, t64 + iu - u,
                  t128 + it - t);
    n += __popcll(mask);
    t64 += __builtin_amdgcn_readlane(iu, 63);
    t128 += __builtin_amdgcn_readlane(it, 63);
    n_big += __popcll(__ballot(mine && r > small_rows));
  }
  if (lane == 0) {
    sched_entry(grp, tiles, (size_t)x * cap + n, -1, 0, 0, t64, t128);
    len[x] = n;
    len[kXcd + 1 + x] = n_big;
  }
}

__global__ __launch_bounds__(1024) void build_sched_kernel(const int32_t* __restrict__ group_off, int n_groups,
                                                           int cap, int4* __restrict__ grp, int2* __restrict__ tiles,
                                                           int* __restrict__ len, int small_rows) {
  const int tid = threadIdx.x;
  if (n_groups <= kSchedSortMax) {
    const int s0 = tid < n_groups ? group_off[tid] : 0;
    build_sched_body(tid < n_groups ? group_off[tid + 1] - s0 : 0, s0, n_groups, cap, grp, tiles, len, small_rows);
  } else if (tid < kXcd) {
    const int x = tid;
    if (x == 0) len[kXcd] = 0;
    int n = 0, t64 = 0, t128 = 0;
    for (int g = x; g < n_groups; g += kXcd) {
      const int s0 = group_off[g], rows = group_off[g + 1] - s0;
      if (rows == 0) continue;
      sched_entry(grp, tiles, (size_t)x * cap + n++, g, s0, rows, t64, t128);
      t64 += (rows + 63) >> 6;
      t128 += (rows + 127) >> 7;
    }
    sched_entry(grp, tiles, (size_t)x * cap + n, -1, 0, 0, t64, t128);
    len[x] = n;
    len[kXcd + 1 + x] = n;   // unsorted lists: no group counts as small (the host passes small_rows = 0 here)
  }
}

// Waits for the vector loads before it, in a form that the compiler takes into account: without it the registers that a
// finder loads now and then would count as on their way at every look-up, each of which would wait for all of the operand
// requests in flight.
__device__ __forceinline__ void finder_loaded() { __builtin_amdgcn_s_waitcnt(0x0F70); }   // vmcnt(0)

// Where the token-major tiles of one XCD lie, out of registers: lane i holds entry i of the XCD's group list, so that a tile
// is found by a ballot.  In memory it is a chain of six dependent scalar loads, a microsecond per tile, which in a launch
// with loader waves stops the operand stream: a contraction of two k tiles (1.7 us) per output tile spent as long on looking
// tiles up as on them.  Lists of more than 63 groups are taken 63 at a time.
struct TileFinder {
  int c, g, slot0, rows;   // lane: tiles before the entry (in m tiles; split lists: of this XCD's, all of them), group, its
                           // first slot, its rows
  uint32_t inv;            // what tile_div divides by the entry's m tiles with
  int b, n, x, tn;
  bool split;
  template <int TM>
  __device__ __forceinline__ void init(const TokenSched& s, int xcd, int n_tiles_n, bool big_only) {
    x = xcd; tn = n_tiles_n; b = 0;
    n = as_const(s.len)[big_only ? kXcd + 1 + x : x];
    split = as_const(s.len)[kXcd] != 0;
    load<TM>(s);
    if (split) {   // at most 7 groups
      const int mine = (int)(threadIdx.x & 63) < n ? share((rows + TM - 1) / TM) : 0;
      c = wave_incl_scan(mine) - mine;
    }
  }
  // tiles of a group of m x tn that are this XCD's (split lists: x, x + 8, ...)
  __device__ __forceinline__ int share(int m) const { return m * tn > x ? (m * tn - x + kXcd - 1) / kXcd : 0; }
  template <int TM>
  __device__ __forceinline__ void load(const TokenSched& s) {
    static_assert(TM == 64 || TM == 128, "the lists hold prefixes of tiles of 64 and of 128 rows");
    // (No branch in here differs per lane: the compiler would fold it into the look-up's loop, take the tile for a value
    // that differs per lane, and issue every operand request from a loop over the lanes.)
    const int i = min(b + (int)(threadIdx.x & 63), s.cap - 1);
    const int4 e = s.grp[(size_t)x * s.cap + i];
    const int2 t = s.tiles[(size_t)x * s.cap + i];
    g = e.x; slot0 = e.y; rows = e.z;
    c = TM == 64 ? t.x : t.y;
    finder_loaded();
    inv = tile_div_inverse((uint32_t)max((rows + TM - 1) / TM, 1));
  }
  // tile number `local` of the XCD (tile ids x, x + 8, ... are numbers 0, 1, ...); false: there is none
  template <int TM>
  __device__ __forceinline__ bool find(const TokenSched& s, int local, int& mt, int& nt, TileCoord& tc) {
    const int lane = threadIdx.x & 63;
    int i, w;
    if (split) {
      const unsigned long long m = __ballot(lane < n && c <= local);
      if (m == 0) return false;
      i = __popcll(m) - 1;
    } else {
      while (b > 0 && local < __builtin_amdgcn_readlane(c, 0) * tn) {   // (a cursor that is behind another one)
        b -= 63;
        load<TM>(s);
      }
      while (n - b > 63 && local >= __builtin_amdgcn_readlane(c, 63) * tn) {
        b += 63;
        load<TM>(s);
      }
      const int here = min(n - b, 63);
      if (here <= 0 || local >= __builtin_amdgcn_readlane(c, here) * tn) return false;
      i = __popcll(__ballot(lane < here && c * tn <= local)) - 1;
    }
    tc.g = __builtin_amdgcn_readlane(g, i);
    tc.slot0 = __builtin_amdgcn_readlane(slot0, i);
    tc.aux = __builtin_amdgcn_readlane(rows, i);
    const int m = (tc.aux + TM - 1) / TM, before = __builtin_amdgcn_readlane(c, i);
    if (split) {
      if (local - before >= share(m)) return false;
      w = x + kXcd * (local - before);
    } else {
      w = local - before * tn;
    }
    nt = tile_div(w, m, (uint32_t)__builtin_amdgcn_readlane((int)inv, i));
    mt = w - nt * m;
    return true;
  }
};

// The same for the neuron-major tiles, of which every group has tm x tn: lane i holds entry b + i of the list.
struct GroupFinder {
  int g, slot0, rows;      // lane: group, its first slot, its rows
  int b, n, x, tm, per;    // tiles of a group on this XCD
  uint32_t inv_per, inv_tm;
  bool split;
  __device__ __forceinline__ void init(const TokenSched& s, int xcd, int tiles_m, int tiles_n, bool big_only) {
    x = xcd; tm = tiles_m; b = 0;
    n = as_const(s.len)[big_only ? kXcd + 1 + x : x];
    split = as_const(s.len)[kXcd] != 0;   // this XCD takes the tiles x, x + 8, ... of every group
    const int all = tiles_m * tiles_n;
    per = !split ? all : all > x ? (all - x + kXcd - 1) / kXcd : 0;
    inv_per = tile_div_inverse((uint32_t)max(per, 1));
    inv_tm = tile_div_inverse((uint32_t)tm);
    load(s);
  }
  __device__ __forceinline__ void load(const TokenSched& s) {
    const int4 e = s.grp[(size_t)x * s.cap + min(b + (int)(threadIdx.x & 63), s.cap - 1)];
    g = e.x; slot0 = e.y; rows = e.z;
    finder_loaded();
  }
  __device__ __forceinline__ bool find(const TokenSched& s, int local, int& mt, int& nt, TileCoord& tc) {
    if (per == 0) return false;
    const int gi = tile_div(local, per, inv_per);
    if (gi >= n) return false;
    if (gi < b || gi >= b + 64) { b = gi & ~63; load(s); }
    int w = local - gi * per;
    if (split) w = x + kXcd * w;
    nt = tile_div(w, tm, inv_tm);
    mt = w - nt * tm;
    tc.g = __builtin_amdgcn_readlane(g, gi - b);
    tc.slot0 = __builtin_amdgcn_readlane(slot0, gi - b);
    tc.aux = __builtin_amdgcn_readlane(rows, gi - b);
    return true;
  }
};

}  // namespace meft
