// Grouped bf16 GEMM on 256 x 256 x 64 tiles: the same contractions, policies and bits as gemm_mfma_kernel, for problems whose
// operands buffer loads reach and whose groups fill such tiles.
//
// What bounds a contraction on gfx950 is how steadily its operands come: a compute unit takes 64 KB per k tile out of L2, and
// at the moment when the tiles that share a panel ask for it every one of them sees the latency of HBM.  So the kernel is
// written for look-ahead.  Four waves, one per SIMD with all of its 512 registers: a wave owns 128 x 128 of the output (256
// accumulators), as 64 rows out of each half of the tile's rows and 64 columns out of each half of its columns, and works
// through a k tile quadrant by quadrant (A0 B0, A0 B1, A1 B0, A1 B1; 16 matrix instructions each) with the fragments of a whole
// half (64 rows x 64 k, 32 registers) in registers.  While a quadrant runs, the fragments that the next one needs and this one
// does not hold are read: B1, A1, then A0 and B0 of the next k tile.  A stage of LDS (two of 64 KB) is therefore given back
// half by half, before its k tile is done: A0 and B0 at the k tile's beginning, A1 and B1 in its middle, and the operands
// requested into it are those of two k tiles later, three quarters of which are still ahead when they have to be there: 96 KB in
// flight per compute unit and 3000 matrix-core cycles of look-ahead out of 128 KB of LDS, where whole stages give 64 KB and 1500.
// A fragment is read once for 128 rows or columns of the other operand, not 64: half the LDS reads per flop of 64 x 128 waves.
// Two barriers per k tile; loads are awaited by count (the 16 most recent ones of a wave may be on their way).
//
// The k tiles of all the tiles of a workgroup form one stream, as in gemm_mfma_kernel.  The stream is the same whatever the tile:
// 16 loads per wave and position, with addresses outside the buffers (zeros, no traffic) for the second half of a tile of at
// most 128 rows and beyond the stream's end.  Loads are issued from asm (they have no output registers): the compiler, which
// cannot tell the halves of a stage apart, would put every LDS read it knows of behind all loads it knows of.
//
// A tile of at most 128 rows (the end of a group) skips the two quadrants of A1: it costs half.  Such tiles come after the
// whole ones in each XCD's order, so that the last round is one of short tiles.
#pragma once
#include "gemm_mfma.h"
#include "tile_share.h"

namespace meft {

constexpr int kWideM = 256;
constexpr int kWideRegion = 128 * kTK * 2;              // 16 KB: 128 rows or columns of one operand, 64 k
constexpr int kWideStage = 4 * kWideRegion;             // A0, A1, B0, B1
constexpr int kWideTurn = 4096;                         // a wave's piece of the output, on its way from columns to rows (two)
constexpr int kWideLds = 2 * kWideStage + 4 * 2 * kWideTurn;

// Where the tiles of one XCD lie: of up to 63 groups at a time the whole tiles (256 rows, more than 128 of them the group's) first,
// then the short ones (a group's last rows, at most 128).  Inside a group the m tiles vary fastest.  Lists that every XCD holds
// (fewer groups than XCDs) are numbered through and dealt in consecutive parts (tile_share.h), the short tiles from the other end:
// an XCD with one whole tile more than others then has none of the short ones left over.
struct WideFinder {
  int g, slot0, rows;            // lane: group, its first slot, its rows
  int nf, cf, ch;                // lane: whole m tiles; whole and short tiles before the entry, from this XCD's first one on
  uint32_t inv;                  // what tile_div divides by nf with
  int b, n, x, base, tn, all_f, all_h;
  __device__ __forceinline__ void init(const TokenSched& s, int xcd, int n_tiles_n, bool big_only) {
    x = xcd; b = 0; base = 0; tn = n_tiles_n;
    n = as_const(s.len)[big_only ? kXcd + 1 + x : x];
    load(s);
    if (as_const(s.len)[kXcd] != 0) {   // every XCD's list is this one: at most seven groups, loaded once
      const int at_f = tile_share_first(all_f, x), at_h = tile_share_first(all_h, kXcd - 1 - x);
      all_f = tile_share_first(all_f, x + 1) - at_f;
      all_h = tile_share_first(all_h, kXcd - x) - at_h;
      cf -= at_f; ch -= at_h;
    }
  }
  __device__ __forceinline__ int live() const {
    const int lane = threadIdx.x & 63;
    return lane < 63 && b + lane < n ? 1 : 0;
  }
  __device__ __forceinline__ void load(const TokenSched& s) {   // (no branch that differs per lane: see TileFinder::load)
    const int i = min(b + (int)(threadIdx.x & 63), s.cap - 1);
    const int4 e = s.grp[(size_t)x * s.cap + i];
    g = e.x; slot0 = e.y; rows = e.z;
    finder_loaded();
    nf = (rows + 127) >> 8;
    const int f = live() * nf * tn, h = rows > nf * kWideM ? live() * tn : 0;
    inv = tile_div_inverse((uint32_t)max(nf, 1));
    cf = wave_incl_scan(f); ch = wave_incl_scan(h);
    all_f = __builtin_amdgcn_readlane(cf, 63);
    all_h = __builtin_amdgcn_readlane(ch, 63);
    cf -= f; ch -= h;
  }
  // tile number `local` of the XCD: its first row, its n tile, and tc.g, tc.slot0, tc.aux = tc.Mrows = the group's rows;
  // false: there is none
  __device__ __forceinline__ bool find(const TokenSched& s, int local, int& m0, int& nt, TileCoord& tc) {
    if (local < base) { b = 0; base = 0; load(s); }   // (a cursor that is behind another one)
    while (local >= base + all_f + all_h) {
      if (b + 63 >= n) return false;
      base += all_f + all_h;
      b += 63;
      load(s);
    }
    const int l = local - base;
    const bool whole = l < all_f;
    const int at = whole ? l : l - all_f;
    // the last entry that begins at or before the tile (one without tiles begins where the next one does, or behind the last)
    const int i = __popcll(__ballot((whole ? cf : ch) <= at && live() != 0)) - 1;
    tc.g = __builtin_amdgcn_readlane(g, i);
    tc.slot0 = __builtin_amdgcn_readlane(slot0, i);
    tc.aux = __builtin_amdgcn_readlane(rows, i);
    const int f = __builtin_amdgcn_readlane(nf, i), w = at - __builtin_amdgcn_readlane(whole ? cf : ch, i);
    nt = whole ? tile_div(w, max(f, 1), (uint32_t)__builtin_amdgcn_readlane((int)inv, i)) : w;
    m0 = (whole ? w - nt * f : f) * kWideM;
    tc.Mrows = tc.aux;
    return true;
  }
};

// A value that is the same in all lanes, for the compiler's eyes: what a loop carries along counts as different per lane
// as soon as one step of the loop looks so.
__device__ __forceinline__ int same(int v) { return __builtin_amdgcn_readfirstlane(v); }

// One 16-byte-per-lane load into LDS at `lds` + `at` (a literal) (a wave's lanes fill 1 KB in order).  M0 wants one wait state before
// the load, and it has it.  A scalar register that a vector instruction has written (v_readlane of a spilled descriptor, say) wants
// five, which the compiler does not look for in front of an asm block.  They are not in here: sixteen loads per k tile with
// three states more each cost the weight gradients 3 to 5 % (17 blocks of 928 x 1088 85.6 / 90.0 us, step of 8192 tokens, 64 blocks of
// 1024 x 4096 2041 / 2072).  tests/test_wait_states.py reads every such load of the built library instead.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"   // (M0 is reserved: nothing of the compiler's outlives a statement in it)
__device__ __forceinline__ void wide_load(i32x4 rsrc, uint32_t voff, int soff, int lds, int at) {
  asm volatile("s_add_i32 m0, %3, %4\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds" ::"v"(voff), "s"(rsrc), "s"(same(soff)),
               "s"(same(lds)), "i"(at)
               : "m0", "scc");
}
#pragma clang diagnostic pop

// A policy is one of gemm_mfma_kernel's, or one with kTM == kWideM, whose locate() deals in tiles of 256 rows; the operands are
// within reach of buffer loads.
#define MEFT_INLINE __attribute__((always_inline))   // of a lambda: one that stays a call keeps what it captures in memory
template <class P>
__global__ __launch_bounds__(256, 1) void gemm_wide_kernel(P p, int n_tiles_bound) {
  static_assert(P::kTM == kWideM, "tiles of 256 rows");
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  typename P::Finder finder = p.finder(blockIdx.x & (kXcd - 1));
  auto next_tile = [&](int wg, TileCoord& t) MEFT_INLINE -> bool {
    if (wg >= n_tiles_bound) return false;
    TileCoord n = t;
    const bool there = same(p.locate(finder, wg, n) ? 1 : 0) != 0;
    t.g = same(n.g); t.m0 = same(n.m0); t.n0 = same(n.n0); t.Mrows = same(n.Mrows);
    t.Ncols = same(n.Ncols); t.nk = same(n.nk); t.slot0 = same(n.slot0); t.aux = same(n.aux);
    return there;
  };
  const int step = gridDim.x;
  constexpr uint32_t kNowhere = 0xFFFFFFF0u;   // offset outside every buffer: such a load brings zeros
  constexpr uint32_t kNoCol = 1u;              // instead of a column's offset (always even): nothing to load
  TileCoord tc;
  if (!next_tile(blockIdx.x, tc)) return;   // the same answer in every wave

  const auto* lds0 = (const __attribute__((address_space(3))) char*)(__attribute__((address_space(3))) void*)smem;
  const uint32_t lds_base = (uint32_t)(uintptr_t)lds0;
  auto make_rsrc = [](const uint16_t* base, uint32_t bytes) {
    const uint64_t a = reinterpret_cast<uint64_t>(base);
    return i32x4{__builtin_amdgcn_readfirstlane((int)(uint32_t)a), __builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32)),
                 __builtin_amdgcn_readfirstlane((int)bytes), 0x00020000};
  };
  const i32x4 rsrc_a = make_rsrc(p.a_base(), p.a_bytes), rsrc_b = make_rsrc(p.b_base(), p.b_bytes);

  // ---------------------------------------------------------------------- operand requests
  // Each wave requests a quarter of every region: its four loads cover, k-contiguous, rows 32 wave + 8 i + lane / 8 (128 bytes
  // of each), otherwise k rows 16 wave + 4 i + lane / 16 (256 bytes of each).
  const int lr8 = lane >> 3, lk = lane >> 4;
  struct Cursor { int wg, k, ok; TileCoord t; } cu{(int)blockIdx.x, 0, 1, tc};
  const int req_base = same((int)lds_base + wave * 4096);
  int req_lds = req_base, req_k = 0;   // this wave's part of the stage that is filled; bytes of the k tiles before
  // lane offsets of the tile's rows (k-contiguous), or of its columns (one for each half)
  constexpr int NA = P::kAMC ? 1 : 4, NB = P::kBNC ? 1 : 4;
  uint32_t oa[2][NA], ob[2][NB];
  [[maybe_unused]] uint32_t ka[4], kb[4];       // n- and m-contiguous operands: row offsets of the position's k rows
  [[maybe_unused]] int ids[16] = {};               // gathered B rows: numbers of this wave's k rows of the next position
  // Which half of its rows (columns) a tile works on first.  The tiles that share a panel run at the same time: every other one
  // of them begins with the second half, so that a line has been on its way for half a k tile when the others ask for it, and
  // each tile waits for memory on one half of its operands only.
  auto swap_a = [](const TileCoord& t) { return t.Mrows - t.m0 > 128 ? (t.n0 >> 8) & 1 : 0; };
  auto swap_b = [](const TileCoord& t) { return (t.m0 >> 8) & 1; };
  auto id_of_row = [&](const int32_t* ids8) MEFT_INLINE -> int {
    const auto* q = as_const(ids8);
    int s[8];
#pragma unroll
    for (int z = 0; z < 8; ++z) s[z] = q[z];
    const int s01 = (lr8 & 1) ? s[1] : s[0], s23 = (lr8 & 1) ? s[3] : s[2], s45 = (lr8 & 1) ? s[5] : s[4],
              s67 = (lr8 & 1) ? s[7] : s[6];
    const int s03 = (lr8 & 2) ? s23 : s01, s47 = (lr8 & 2) ? s67 : s45;
    return (lr8 & 4) ? s47 : s03;
  };
  auto fetch_ids = [&]() MEFT_INLINE {   // of position cu
    if constexpr (P::kBNC) {
      if constexpr (P::kRowIdsInMemory) {
        if (cu.ok) {
          const auto* q = as_const(p.b_row_id_src(cu.t, cu.k * kTK) + wave * 16);
#pragma unroll
          for (int z = 0; z < 16; ++z) ids[z] = q[z];
        }
      }
    }
  };
  auto setup = [&]() MEFT_INLINE {
    const TileCoord& t = cu.t;
    const int chunk = (lane & 15) ^ (4 * (lk & 3));
    const int sa = swap_a(t) << 7, sb = swap_b(t) << 7;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int ha = (h << 7) ^ sa, hb = (h << 7) ^ sb;   // first row or column of the half
      if constexpr (P::kAMC) {
        const int col = t.m0 + ha + chunk * 8, last = p.a_cols(t) - 8;
        oa[h][0] = cu.ok ? byte_off(p.a_mat() + (col > last ? last : col), p.a_base()) : kNoCol;
        if (h == 1 && t.Mrows - t.m0 <= 128) oa[h][0] = kNoCol;
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int r8 = ha + wave * 32 + i * 8, row = r8 + lr8;
          int id = 0, m = t.m0 + row;
          const bool there = cu.ok && m < t.Mrows;
          m = m < t.Mrows ? m : t.Mrows - 1;
          if constexpr (P::kAIds) id = id_of_row(p.a_ids(t) + min(r8, t.Mrows - t.m0 - 1));
          const uint32_t o = byte_off(p.a_row(t, m, id), p.a_base()) + (uint32_t)(((lane & 7) ^ ((row >> 1) & 7)) << 4);
          oa[h][i] = there ? o : kNowhere;
        }
      }
      if constexpr (P::kBNC) {
        const int col = t.n0 + hb + chunk * 8;
        ob[h][0] = cu.ok && col < t.Ncols ? byte_off(p.b_row_ptr(0) + col, p.b_base()) : kNoCol;
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int r8 = hb + wave * 32 + i * 8, row = r8 + lr8, n = min(t.n0 + row, t.Ncols - 1);
          int from = n, there = cu.ok && t.n0 + row < t.Ncols ? 1 : 0;
          if constexpr (P::kBTags) {
            const int tag = id_of_row(p.b_tags(t) + r8);
            there &= tag > 0 ? 1 : 0;
            from = max(tag, 1) - 1;
          }
          const uint32_t o = byte_off(p.b_row(t, from), p.b_base()) + (uint32_t)(((lane & 7) ^ ((row >> 1) & 7)) << 4);
          ob[h][i] = there ? o : kNowhere;
        }
      }
    }
  };
  // the offsets of the position's k rows
  auto position = [&]() MEFT_INLINE {
    const TileCoord& t = cu.t;
    if constexpr (P::kAMC) {
      const uint32_t row_bytes = (uint32_t)p.a_cols(t) * 2u;
#pragma unroll
      for (int i = 0; i < 4; ++i) ka[i] = (uint32_t)p.a_krow(t, cu.k * kTK + wave * 16 + i * 4 + lk) * row_bytes;
    }
    if constexpr (P::kBNC) {
      const uint32_t row_bytes = (uint32_t)t.Ncols * 2u;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        int id;
        if constexpr (P::kRowIdsInMemory) {
          const int s01 = (lk & 1) ? ids[4 * i + 1] : ids[4 * i], s23 = (lk & 1) ? ids[4 * i + 3] : ids[4 * i + 2];
          id = (lk & 2) ? s23 : s01;
        } else {
          id = p.b_row_ids(t, cu.k * kTK + wave * 16 + i * 4 + lk);
        }
        kb[i] = (uint32_t)id * row_bytes;
      }
    }
  };
  auto request_a = [&](int h, int i) MEFT_INLINE {
    const int at = h * kWideRegion + i * 1024;
    if constexpr (P::kAMC) wide_load(rsrc_a, oa[h][0] == kNoCol ? kNowhere : oa[h][0] + ka[i], 0, req_lds, at);
    else wide_load(rsrc_a, oa[h][i], req_k, req_lds, at);
  };
  auto request_b = [&](int h, int i) MEFT_INLINE {
    const int at = (2 + h) * kWideRegion + i * 1024;
    if constexpr (P::kBNC) wide_load(rsrc_b, ob[h][0] == kNoCol ? kNowhere : ob[h][0] + kb[i], 0, req_lds, at);
    else wide_load(rsrc_b, ob[h][i], req_k, req_lds, at);
  };
  auto advance = [&]() MEFT_INLINE {
    req_lds = same(req_base + (req_base + kWideStage - req_lds));   // the other stage
    cu.k = same(cu.k + 1);
    req_k = same(req_k + kTK * 2);
    if (same(cu.ok != 0 && cu.k == cu.t.nk ? 1 : 0)) {
      cu.wg = same(cu.wg + step);
      cu.k = 0; req_k = 0;
      cu.ok = same(next_tile(cu.wg, cu.t) ? 1 : 0);
      setup();
    }
    fetch_ids();
  };

  // ---------------------------------------------------------------------- fragments
  const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;
  const int fr = lane & 31, fc = lane >> 5;
  // byte offsets inside a region: k-contiguous one per k16 step (fragment i is 32 rows = 4096 bytes on), otherwise one per
  // fragment (a k16 step is 4096 bytes on, the high k half 1024)
  uint32_t ra[4], rb[4];
  {
    const int gq = lane >> 4, s = lane & 15, k_lo = 8 * (gq >> 1) + (s >> 2);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if constexpr (P::kAMC) {
        const int m = wm + (q & 1) * 32 + 16 * (gq & 1) + 4 * (s & 3);
        ra[q] = (uint32_t)(k_lo * 128 + (((m >> 3) ^ (4 * (k_lo & 3))) << 3) + (m & 7)) * 2u;
      } else {
        ra[q] = (uint32_t)((wm + fr) * 128 + (((q * 2 + fc) ^ ((fr >> 1) & 7)) << 4));
      }
      if constexpr (P::kBNC) {
        const int n = wn + (q & 1) * 32 + 16 * (gq & 1) + 4 * (s & 3);
        rb[q] = (uint32_t)(k_lo * 128 + (((n >> 3) ^ (4 * (k_lo & 3))) << 3) + (n & 7)) * 2u;
      } else {
        rb[q] = (uint32_t)((wn + fr) * 128 + (((q * 2 + fc) ^ ((fr >> 1) & 7)) << 4));
      }
    }
  }
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  typedef short s16x8 __attribute__((ext_vector_type(8)));
  struct Half { bf16x8 f[4][2]; };   // [k16 step][fragment]
  Half A0, A1, B0, B1;
  auto read1 = [&](auto tr_tag, Half& to, int ks, int i, uint32_t region, const uint32_t (&r)[4]) MEFT_INLINE {
    constexpr bool kTr = decltype(tr_tag)::value;
    if constexpr (kTr) {
      const auto* q = lds0 + (region + r[i] + ks * 4096);
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(q));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(q + 1024));
      to.f[ks][i] = __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    } else {
      to.f[ks][i] = *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>(lds0 + (region + r[ks] + i * 4096));
    }
  };
  using TrA = std::integral_constant<bool, P::kAMC>;
  using TrB = std::integral_constant<bool, P::kBNC>;
  uint32_t stage = 0;   // of the position that is worked on, in bytes
  auto read_a = [&](Half& to, uint32_t st, int h, int ks, int i) MEFT_INLINE { read1(TrA{}, to, ks, i, st + h * kWideRegion, ra); };
  auto read_b = [&](Half& to, uint32_t st, int h, int ks, int i) MEFT_INLINE { read1(TrB{}, to, ks, i, st + (2 + h) * kWideRegion, rb); };

#define MEFT_FENCE() __builtin_amdgcn_sched_barrier(0)
  // The 16 matrix instructions of one quadrant; after instruction z (of 16) comes extra(z).
  auto quadrant = [&](auto zero_tag, auto ah_tag, auto bh_tag, auto& acc, const Half& a, const Half& b, auto&& extra) MEFT_INLINE {
    constexpr bool kZero = decltype(zero_tag)::value;
    constexpr int ah = decltype(ah_tag)::value, bh = decltype(bh_tag)::value;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          f32x16& c = acc[ah * 2 + i][bh * 2 + j];
          if (kZero && ks == 0) {
            const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b.f[ks][j], a.f[ks][i], zero, 0, 0, 0);
          } else {
            c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b.f[ks][j], a.f[ks][i], c, 0, 0, 0);
          }
          MEFT_FENCE();
          extra(ks * 4 + i * 2 + j);
          MEFT_FENCE();
        }
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  // Barrier: this wave's LDS reads have returned, and (awaited) of its loads only the 16 most recent are on their way.
  auto barrier = [&](bool awaited) MEFT_INLINE {
    if (awaited) asm volatile("s_waitcnt vmcnt(16) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    else asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  };
  // What goes between a quadrant's matrix instructions: a request after every fourth, eight fragment reads between those, the
  // last of them early enough to be back at a barrier.
  auto is_request = [](int z) { return (z & 3) == 3; };
  auto is_read = [](int z) { return (z & 3) != 3 && z < 10; };
  auto read_no = [](int z) { return z - (z >> 2); };
  // One k tile.  wait: false for a tile's first one, whose operands were awaited before the stores of the tile before: those
  // have half a k tile to leave before a barrier waits for them.
  auto k_tile = [&](auto zero_tag, auto short_tag, auto& acc, bool wait) MEFT_INLINE {
    constexpr bool kShort = decltype(short_tag)::value;
    const uint32_t next = stage ^ kWideStage;
    barrier(wait);   // A0 and B0 of this position are in every wave's registers, A1 and B1 have landed
    quadrant(zero_tag, I0{}, I0{}, acc, A0, B0, [&](int z) MEFT_INLINE {
      if (is_read(z)) read_b(B1, stage, 1, read_no(z) >> 1, read_no(z) & 1);
      if (z == 2) position();
      if (is_request(z)) request_a(0, z >> 2);
      if constexpr (kShort) { if (is_request(z)) request_b(0, z >> 2); }
    });
    if constexpr (!kShort) {
      quadrant(zero_tag, I0{}, I1{}, acc, A0, B1, [&](int z) MEFT_INLINE {
        if (is_read(z)) read_a(A1, stage, 1, read_no(z) >> 1, read_no(z) & 1);
        if (is_request(z)) request_b(0, z >> 2);
      });
    }
    barrier(true);   // A1 and B1 are in every wave's registers, A0 and B0 of the next position have landed
    if constexpr (kShort) {
      quadrant(zero_tag, I0{}, I1{}, acc, A0, B1, [&](int z) MEFT_INLINE {
        if (is_read(z)) read_b(B0, next, 0, read_no(z) >> 1, read_no(z) & 1);
        if ((z & 3) == 3) { read_a(A0, next, 0, z >> 2, 0); read_a(A0, next, 0, z >> 2, 1); }   // (their last use is behind)
        if (is_request(z)) { request_a(1, z >> 2); request_b(1, z >> 2); }
      });
    } else {
      quadrant(zero_tag, I1{}, I0{}, acc, A1, B0, [&](int z) MEFT_INLINE {
        if (is_read(z)) read_a(A0, next, 0, read_no(z) >> 1, read_no(z) & 1);
        if (is_request(z)) request_a(1, z >> 2);
      });
      quadrant(zero_tag, I1{}, I1{}, acc, A1, B1, [&](int z) MEFT_INLINE {
        if (is_read(z)) read_b(B0, next, 0, read_no(z) >> 1, read_no(z) & 1);
        if (is_request(z)) request_b(1, z >> 2);
      });
    }
    advance();
    MEFT_FENCE();
    stage = next;
  };

  setup();
  fetch_ids();
#pragma unroll 1
  for (int s = 0; s < 2; ++s) {
    position();
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < 4; ++i) { request_a(h, i); request_b(h, i); }
    advance();
  }
  asm volatile("s_waitcnt vmcnt(16)\n\ts_barrier" ::: "memory");

  // One output tile: acc[row half * 2 + i][column half * 2 + j] (a tile of at most 128 rows has no second row half)
  auto tile = [&](auto short_tag) MEFT_INLINE {
    constexpr bool kShort = decltype(short_tag)::value;
    f32x16 acc[kShort ? 2 : 4][4];
    const int sa = swap_a(tc) << 7, sb = swap_b(tc) << 7;
    const int tag0 = p.row_tag(tc, tc.m0 + sa + wm + lane);
    const int tag1 = kShort ? 0 : p.row_tag(tc, tc.m0 + (128 ^ sa) + wm + lane);
    const int nk = tc.nk;
    // (read again where the last k tile of the tile before has read them: they hold no registers during its stores)
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int i = 0; i < 2; ++i) { read_a(A0, stage, 0, ks, i); read_b(B0, stage, 0, ks, i); }
    k_tile(std::true_type{}, short_tag, acc, false);
#pragma unroll 1
    for (int kt = 1; kt < nk; ++kt) k_tile(std::false_type{}, short_tag, acc, true);
    [[maybe_unused]] u32x4 aux[P::kAux ? (kShort ? 2 : 4) * 2 * 4 : 1];
    if constexpr (P::kAux) {
      // all of them at once, into the registers that the fragments leave: behind stores each would wait for those
      static_assert(!P::kAux || P::kOutBf16, "16 bytes are 8 columns");
#pragma unroll
      for (int ri = 0; ri < (kShort ? 2 : 4); ++ri)
#pragma unroll
        for (int pc = 0; pc < 2; ++pc)
#pragma unroll
          for (int t = 0; t < 4; ++t)
            aux[(ri * 2 + pc) * 4 + t] = p.load_aux16(tc, tc.m0 + wm + (((ri >> 1) << 7) ^ sa) + (ri & 1) * 32 + (lane >> 3) + 8 * t,
                                                      tc.n0 + wn + ((pc << 7) ^ sb) + (lane & 7) * 8);
    }
    // the next tile's first position has landed before this one's stores
    asm volatile("s_waitcnt vmcnt(16)" ::: "memory");

    // ---- epilogue.  The matrix instructions were handed B first: lane l holds, of row m = l % 32 of a fragment, the columns
    // n = 8 (r / 4) + 4 (l / 32) + r % 4, four at a time side by side.  Pieces of 32 rows x 128 bytes (64 columns of bf16, 32 of
    // fp32) turn in LDS, in the wave's own 8 KB, two pieces by turns: then a lane holds 16 consecutive bytes, and a store covers
    // 8 rows x 128 bytes.  (With two columns per lane, out of the registers through neighbour swaps, the epilogue was 2000 vector
    // instructions and 128 to 512 stores per wave, as long as ten k tiles.)
    {
      const auto* turn = lds0 + 2 * kWideStage + wave * 2 * kWideTurn;
      auto* turn_w = (__attribute__((address_space(3))) char*)turn;
      const int trow = lane >> 3, tchunk = lane & 7;           // of the row-wise side
      constexpr int kCols = P::kOutBf16 ? 64 : 32;             // columns of a piece
      constexpr int kPieces = P::kOutBf16 ? 2 : 4;             // pieces of a wave's 128 columns
      constexpr int kEach = P::kOutBf16 ? 8 : 4;               // columns of 16 bytes
      const int ocols = p.out_cols(tc);
      const int ncol = tc.n0 + wn + tchunk * kEach;
      [[maybe_unused]] size_t lane_at = 0;
      [[maybe_unused]] int ld = 0;
      if constexpr (P::kRowsLinear) {
        ld = p.out_ld(tc);
        lane_at = p.row_off(tc, 1, tc.m0 + wm + trow) + ncol;
      }
      const unsigned long long ok0 = __ballot(tag0 != 0), ok1 = __ballot(tag1 != 0);
      // columns to rows: the piece's values into LDS ...
      auto put = [&](int ri, int pc, int buf) MEFT_INLINE {
        auto* to = turn_w + buf * kWideTurn + (lane & 31) * 128;
        const int key = ((lane & 31) >> 1) & 7;
        if constexpr (P::kOutBf16) {
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            // (they stay accumulation registers up to here: copied to vector registers any earlier, all pieces' would not fit)
            f32x16 c = acc[ri][pc * 2 + j];
            asm volatile("" : "+a"(c));
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const u32x2 v = {pack_bf16x2(c[4 * q], c[4 * q + 1]), pack_bf16x2(c[4 * q + 2], c[4 * q + 3])};
              *reinterpret_cast<__attribute__((address_space(3))) u32x2*>(to + (((j * 4 + q) ^ key) << 4) + fc * 8) = v;
            }
          }
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const f32x16& c = acc[ri][pc];
            const f32x4 v = {c[4 * q], c[4 * q + 1], c[4 * q + 2], c[4 * q + 3]};
            *reinterpret_cast<__attribute__((address_space(3))) f32x4*>(to + (((q * 2 + fc) ^ key) << 4)) = v;
          }
        }
      };
      // ... and out of it into memory
      auto get = [&](int ri, int pc, int buf) MEFT_INLINE {
        const int col = pc * kCols >= 64 ? (128 ^ sb) + pc * kCols - 64 : sb + pc * kCols;   // first column, of the wave's
        if (tc.n0 + wn + col >= ocols) return;
        int row0 = (((ri >> 1) << 7) ^ sa) + (ri & 1) * 32;
        asm volatile("" : "+s"(row0));   // (addresses worked out ahead of the stores would not fit the registers)
        u32x4 v[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int row = trow + 8 * t;
          v[t] = *reinterpret_cast<const __attribute__((address_space(3))) u32x4*>(turn + buf * kWideTurn + row * 128 +
                                                                                  ((tchunk ^ ((row >> 1) & 7)) << 4));
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int rl = (ri & 1) * 32 + trow + 8 * t;   // of the wave's 64 rows of this half
          int tag;
          if constexpr (P::kRowsLinear) tag = (int)(((ri < 2 ? ok0 : ok1) >> rl) & 1ull);
          else tag = __builtin_amdgcn_ds_bpermute(rl << 2, ri < 2 ? tag0 : tag1);
          if (tag != 0) {
            size_t at;
            if constexpr (P::kRowsLinear) at = lane_at + (size_t)((row0 + 8 * t) * ld + col);
            else at = p.row_off(tc, tag, tc.m0 + wm + row0 + trow + 8 * t) + ncol + col;
            if constexpr (P::kAux) p.store16(at, ncol + col, v[t], aux[(ri * 2 + pc) * 4 + t]);
            else p.store16(at, ncol + col, v[t], u32x4{0u, 0u, 0u, 0u});
          }
        }
      };
      constexpr int kAll = (kShort ? 2 : 4) * kPieces;
#pragma unroll
      for (int z = 0; z <= kAll; ++z) {
        if (z < kAll) put(z / kPieces, z % kPieces, z & 1);
        asm volatile("" ::: "memory");   // (what a lane reads, another has written: the order stands, a wave's LDS traffic keeps it)
        if (z > 0) get((z - 1) / kPieces, (z - 1) % kPieces, (z - 1) & 1);
        asm volatile("" ::: "memory");
        MEFT_FENCE();
      }
    }
  };

  for (int wg = blockIdx.x;;) {
    if (tc.Mrows - tc.m0 <= 128) tile(std::true_type{});
    else tile(std::false_type{});
    wg += step;
    if (!next_tile(wg, tc)) break;
  }
#undef MEFT_FENCE
#undef MEFT_INLINE
  // no load may land in LDS that has gone to another workgroup
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

}  // namespace meft
