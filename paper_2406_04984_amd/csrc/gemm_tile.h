// Small-tile form of the grouped bf16 contraction (gemm_mfma.h has the problem statement, the LDS swizzles' reasons and
// the tile schedule): tiles of TM x TN x 64, four waves as 2 x 2, every wave requests a quarter of the operands itself
// through buffer loads into LDS, three slots per operand.
//
// For the token-major problems whose 128 x 256 tiles do not fill the chip (groups of around a hundred tokens, blocks of a
// few hundred neurons): there a compute unit works through one tile and its time is the time the tile's operands take
// into LDS, about 1 us per 48 KB k tile (a compute unit has about a hundred 128-byte lines in flight), while half the
// chip idles, and a block of fewer than 256 neurons still loads 256 rows.  A 64 x 128 tile brings at most 24 KB per k
// tile, leaves room for a second workgroup on the compute unit (72 KB each) whose work passes under this one's waits, and
// there are four times as many.  Key scores 32.6 -> 19.2 us and activation gradient 29.5 -> 16.9 us at 1589 tokens x 2
// blocks of 29 x 336, d 1792; 54 -> 45 and 57 -> 43 us at 2003 x 8 of 64 x 96, d 4096.  Where large tiles do fill the chip
// they move fewer bytes per flop and win (value sum of the latter: 52 against 71 us).
//
// Schedule of one k tile (four k16 steps):
//   step 0..2   matrix instructions of the step, then the LDS reads of the step after it, whose latency passes under them
//   wait        own requests of the next k tile (the ones of the k tile after that may be on their way); barrier:
//               everyone is past this k tile's slot (every LDS read has been waited for where it was issued), and the
//               next k tile's has landed
//   step 3      matrix instructions, the requests of the k tile three ahead into the slot just released, LDS reads of
//               the next k tile's step 0
// The requests run on across tiles.  Fragment reads are asm: through builtins the compiler orders every LDS read behind
// all outstanding global -> LDS loads.
// A request never branches: what must not be read (rows beyond the group, contraction indices beyond the end, a k tile
// beyond the stream) gets an offset outside the buffer, which loads zeros without touching memory.
#pragma once
#include "gemm_mfma.h"

namespace meft {

#define MEFT_LOAD_LDS16(rsrc, voff, soff, dst) \
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, MEFT_LPTR(dst), 16, (int)(voff), (int)(soff), 0, 0)

template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (N > 0) {
    static_for<N - 1>(f);
    f(std::integral_constant<int, N - 1>{});
  }
}

// The LDS reads of one k16 step (one A fragment, two B fragments) with the wait for them, in one asm statement: through
// builtins the compiler orders every LDS read behind all outstanding global -> LDS loads, and the outputs of a read
// without its wait would count as written while they are on their way.
template <int OFFA, int OFFB0, int OFFB1>
__device__ __forceinline__ void lds_read_kc3(u32x4& a, u32x4& b0, u32x4& b1, uint32_t xa, uint32_t xb) {
  asm volatile(
      "ds_read_b128 %0, %3 offset:%5\n\t"
      "ds_read_b128 %1, %4 offset:%6\n\t"
      "ds_read_b128 %2, %4 offset:%7\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(a), "=&v"(b0), "=&v"(b1)
      : "v"(xa), "v"(xb), "n"(OFFA), "n"(OFFB0), "n"(OFFB1)
      : "memory");
}
// the B fragments by transposing reads, low and high k half each
template <int OFFA, int OFFB>
__device__ __forceinline__ void lds_read_nc3(u32x4& a, u32x2 (&b)[4], uint32_t xa, uint32_t b0lo, uint32_t b0hi, uint32_t b1lo,
                                             uint32_t b1hi) {
  asm volatile(
      "ds_read_b128 %0, %5 offset:%10\n\t"
      "ds_read_b64_tr_b16 %1, %6 offset:%11\n\t"
      "ds_read_b64_tr_b16 %2, %7 offset:%11\n\t"
      "ds_read_b64_tr_b16 %3, %8 offset:%11\n\t"
      "ds_read_b64_tr_b16 %4, %9 offset:%11\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(a), "=&v"(b[0]), "=&v"(b[1]), "=&v"(b[2]), "=&v"(b[3])
      : "v"(xa), "v"(b0lo), "v"(b0hi), "v"(b1lo), "v"(b1hi), "n"(OFFA), "n"(OFFB)
      : "memory");
}

// Chunk swizzle of row k of an operand that is contiguous along its own index, COLS elements per row (chunks of 16 B):
// the sixteen lanes of a transposing read take two chunks of each of four consecutive rows, which this spreads over
// the banks.
template <int COLS>
__device__ __forceinline__ int nc_key(int k) {
  static_assert(COLS == 128, "");
  return 4 * (k & 3);
}

template <class P>
constexpr int gemm_tile_lds() { return 3 * (P::kTM + P::kTNt) * kTK * 2; }

// A policy P provides, besides what gemm_mfma.h asks of it:
//   static constexpr int kTM, kTNt;        64 or 128 rows and columns of a tile
//   __device__ int tiles_n() const;
//   __device__ void coord(int mt, int nt, TileCoord&) const;   m0, n0, Mrows, Ncols, nk from g, slot0, aux (= rows)
//   static constexpr bool kAIds;           false: row m of A is row slot0 + m of a_base();  true: its number is entry m of
//   __device__ const int32_t* a_ids(const TileCoord&) const;   (readable TM entries beyond the group)
//   __device__ int a_ld() const;           row length of A in elements (A is k-contiguous)
//   out_base(), o_bytes;                   the output array (below 4 GB), its rows of an even number of columns
//   uint32_t keep(uint32_t pk, int n, uint32_t aux) const;   bf16 output: what of the two values is stored
//   B k-contiguous: row n is row b_row0() + n of b_base(), n < Ncols;   b_ld()
//   B n-contiguous: row k is row b_row0() + k, k < b_rows()
template <class P>
__global__ __launch_bounds__(256, 2) void gemm_tile_kernel(P p, int n_tiles_bound) {
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];   // three A slots, three B slots
  const int wg0 = blockIdx.x, step = gridDim.x;
  constexpr int TM = P::kTM, TN = P::kTNt;
  constexpr int MI = TM / 64, NJ = TN / 64;                 // 32 x 32 accumulators of a wave
  constexpr int LA = TM / 32, LB = TN / 32, NL = LA + LB;   // 1 KB requests of a wave per k tile
  constexpr int kASlot = TM * kTK, kBSlot = TN * kTK;       // elements
  constexpr uint32_t kNowhere = 0xFFFFFFF0u;
  const __amdgpu_buffer_rsrc_t rsrc_o = __builtin_amdgcn_make_buffer_rsrc(p.out_base(), 0, (int)p.o_bytes, 0x00020000);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  TileFinder fr_, fc_;
  fr_.template init<TM>(p.sched, wg0 & (kXcd - 1), p.tiles_n(), p.big_only != 0);
  fc_ = fr_;
  auto next_tile = [&](TileFinder& f, int wg, TileCoord& t) -> bool {
    int mt, nt;
    if (wg >= n_tiles_bound || !f.template find<TM>(p.sched, wg >> 3, mt, nt, t)) return false;
    p.coord(mt, nt, t);
    return true;
  };
  TileCoord tc;
  if (!next_tile(fc_, wg0, tc)) return;   // the same answer in every wave

  // ---- operand requests ------------------------------------------------------------------------------------------
  const __amdgpu_buffer_rsrc_t rsrc_a = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p.a_base()), 0, (int)p.a_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_b = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p.b_base()), 0, (int)p.b_bytes, 0x00020000);
  const int lr8 = lane >> 3;
  struct { int wg, k; bool ok; TileCoord t; } cu{wg0, 0, true, tc};
  int req = 0;   // slot of the next request
  // k-contiguous: a request covers 8 rows x 128 bytes; one offset per request, the k offset is the instruction's scalar.
  // contiguous along its own index: a request covers R = 512 / COLS contraction rows x 2 COLS bytes; one offset serves all.
  constexpr int RB = 512 / TN;
  uint32_t oa[LA], ob[P::kBNC ? 1 : LB];
  auto setup = [&]() {
    const TileCoord& t = cu.t;
    {
      const uint32_t rb = (uint32_t)p.a_ld() * 2u;
      if constexpr (P::kAIds) {
        const auto* ids = as_const(p.a_ids(t) + wave * (TM / 4));
#pragma unroll
        for (int i = 0; i < LA; ++i) {
          int s[8];
#pragma unroll
          for (int z = 0; z < 8; ++z) s[z] = ids[i * 8 + z];
          const int s01 = (lr8 & 1) ? s[1] : s[0], s23 = (lr8 & 1) ? s[3] : s[2], s45 = (lr8 & 1) ? s[5] : s[4],
                    s67 = (lr8 & 1) ? s[7] : s[6];
          const int s03 = (lr8 & 2) ? s23 : s01, s47 = (lr8 & 2) ? s67 : s45;
          oa[i] = (uint32_t)((lr8 & 4) ? s47 : s03);
        }
      } else {
#pragma unroll
        for (int i = 0; i < LA; ++i) oa[i] = (uint32_t)(t.slot0 + t.m0 + wave * (TM / 4) + i * 8 + lr8);
      }
#pragma unroll
      for (int i = 0; i < LA; ++i) {
        const int row = wave * (TM / 4) + i * 8 + lr8;
        const uint32_t o = oa[i] * rb + ((((lane & 7) ^ ((row >> 1) & 7)) << 3)) * 2u;
        oa[i] = t.m0 + row < t.Mrows ? o : kNowhere;
      }
    }
    if constexpr (P::kBNC) {
      const int row = lane / (TN / 8), col = t.n0 + (((lane % (TN / 8)) ^ nc_key<TN>(row)) << 3);
      // (columns beyond the matrix are not stored)
      ob[0] = (uint32_t)min(col, t.Ncols - 8) * 2u + (uint32_t)row * ((uint32_t)t.Ncols * 2u);
    } else {
#pragma unroll
      for (int i = 0; i < LB; ++i) {
        const int row = wave * (TN / 4) + i * 8 + lr8;
        const uint32_t o = (uint32_t)(p.b_row0(t) + t.n0 + row) * ((uint32_t)p.b_ld() * 2u) + ((((lane & 7) ^ ((row >> 1) & 7)) << 3)) * 2u;
        ob[i] = t.n0 + row < t.Ncols ? o : kNowhere;
      }
    }
  };
  // request number N (A first) of the cursor's k tile
  auto request = [&](auto n_tag) {
    constexpr int N = decltype(n_tag)::value;
    const TileCoord& t = cu.t;
    const int k0 = cu.k * kTK;
    if constexpr (N < LA) {
      uint16_t* dst = smem + req * kASlot + (wave * LA + N) * 512;
      MEFT_LOAD_LDS16(rsrc_a, oa[N], k0 * 2, dst);
    } else {
      constexpr int i = N - LA;
      uint16_t* dst = smem + 3 * kASlot + req * kBSlot + (wave * LB + i) * 512;
      if constexpr (P::kBNC) {
        const uint32_t rb = (uint32_t)t.Ncols * 2u;
        const int kk = k0 + wave * 16 + RB * i, kl = kk + lane / (TN / 8);
        MEFT_LOAD_LDS16(rsrc_b, kl < p.b_rows(t) ? ob[0] : kNowhere, (uint32_t)(p.b_row0(t) + min(kk, p.b_rows(t) - 1)) * rb, dst);
      } else {
        MEFT_LOAD_LDS16(rsrc_b, ob[i], k0 * 2, dst);
      }
    }
  };
  auto advance = [&]() {
    req = req == 2 ? 0 : req + 1;
    if (++cu.k == cu.t.nk) {
      cu.wg += step; cu.k = 0; cu.ok = next_tile(fr_, cu.wg, cu.t);
      if (cu.ok) setup();
    }
    if (!cu.ok) {   // the stream has ended
#pragma unroll
      for (auto& o : oa) o = kNowhere;
#pragma unroll
      for (auto& o : ob) o = kNowhere;
      cu.k = 0;
      cu.t.nk = 0x7FFFFFFF;
    }
  };

  // ---- fragments -------------------------------------------------------------------------------------------------
  const int fr = lane & 31, fc = lane >> 5;
  const int wm = (wave >> 1) * (TM / 2), wn = (wave & 1) * (TN / 2);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)smem;
  const uint32_t ldsb = lds0 + 3u * kASlot * 2u;
  // LDS byte addresses of this lane's fragment reads in slot 0.  k-contiguous: one per k16 step (the swizzle key does not
  // depend on the 32-row fragment); transposing: low / high half per fragment, one for all steps.
  uint32_t xa[4], xb[P::kBNC ? NJ : 4], xbh[P::kBNC ? NJ : 1];
  {
    const int gq = lane >> 4, s = lane & 15;
    const int k_lo = 8 * (gq >> 1) + (s >> 2), k_hi = k_lo + 4;
#pragma unroll
    for (int z = 0; z < 4; ++z)
      xa[z] = lds0 + (uint32_t)((wm + fr) * kTK + (((z * 2 + fc) ^ ((fr >> 1) & 7)) << 3)) * 2u;
    if constexpr (P::kBNC) {
#pragma unroll
      for (int z = 0; z < NJ; ++z) {
        const int n = wn + z * 32 + 16 * (gq & 1) + 4 * (s & 3);
        xb[z] = ldsb + (uint32_t)(k_lo * TN + (((n >> 3) ^ nc_key<TN>(k_lo)) << 3) + (n & 7)) * 2u;
        xbh[z] = ldsb + (uint32_t)(k_hi * TN + (((n >> 3) ^ nc_key<TN>(k_hi)) << 3) + (n & 7)) * 2u;
      }
    } else {
#pragma unroll
      for (int z = 0; z < 4; ++z)
        xb[z] = ldsb + (uint32_t)((wn + fr) * kTK + (((z * 2 + fc) ^ ((fr >> 1) & 7)) << 3)) * 2u;
    }
  }
  struct Frags { u32x4 a[MI], b[NJ]; };
  Frags f0, f1;
  f32x16 acc[MI][NJ];
  int slot = 0;
  static_assert(MI == 1 && NJ == 2, "read_frags");
  auto read_frags = [&](auto ks_tag, Frags& f) {
    constexpr int KS = decltype(ks_tag)::value;
    const uint32_t soa = (uint32_t)slot * (kASlot * 2), sob = (uint32_t)slot * (kBSlot * 2);
    if constexpr (P::kBNC) {
      u32x2 b[4];
      lds_read_nc3<0, KS * 16 * TN * 2>(f.a[0], b, xa[KS] + soa, xb[0] + sob, xbh[0] + sob, xb[1] + sob, xbh[1] + sob);
      f.b[0] = u32x4{b[0].x, b[0].y, b[1].x, b[1].y};
      f.b[1] = u32x4{b[2].x, b[2].y, b[3].x, b[3].y};
    } else {
      lds_read_kc3<0, 0, 32 * kTK * 2>(f.a[0], f.b[0], f.b[1], xa[KS] + soa, xb[KS] + sob);
    }
  };
#define MEFT_FENCE() __builtin_amdgcn_sched_barrier(0)
  auto mma = [&](auto zero_tag, auto j_tag, const Frags& f) {
    constexpr int j = decltype(j_tag)::value;
    const bf16x8 av = __builtin_bit_cast(bf16x8, f.a[0]), bv = __builtin_bit_cast(bf16x8, f.b[j]);
    if constexpr (decltype(zero_tag)::value) {
      const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      acc[0][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bv, zero, 0, 0, 0);
    } else {
      acc[0][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bv, acc[0][j], 0, 0, 0);
    }
    MEFT_FENCE();
  };
#define KS(n) std::integral_constant<int, n> {}
  // f0 holds step 0 of the current k tile; at the end it holds step 0 of the next one (if there is none, stale bytes)
  // The barrier of k tile q waits for the requests of q + 1; those of q + 2 (NL per wave) may be on their way, and in
  // the first two k tiles after a tile's end so may its stores (always kStores per wave), which were issued after them.
  constexpr int kStores = 8 * MI * NJ;
  int since = 2;   // k tiles since the last stores
  auto k_tile = [&](auto first) {
    mma(first, KS(0), f0); mma(first, KS(1), f0); read_frags(KS(1), f1); MEFT_FENCE();
    mma(std::false_type{}, KS(0), f1); mma(std::false_type{}, KS(1), f1); read_frags(KS(2), f0); MEFT_FENCE();
    mma(std::false_type{}, KS(0), f0); mma(std::false_type{}, KS(1), f0); read_frags(KS(3), f1); MEFT_FENCE();
    if (since < 2) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(NL + kStores) : "memory");
    else asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(NL) : "memory");
    ++since;
    MEFT_FENCE();
    slot = slot == 2 ? 0 : slot + 1;
    mma(std::false_type{}, KS(0), f1);
    static_for<NL>([&](auto n) { request(n); });
    MEFT_FENCE();
    mma(std::false_type{}, KS(1), f1);
    advance();
    read_frags(KS(0), f0);
    MEFT_FENCE();
  };

  setup();
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    static_for<NL>([&](auto n) { request(n); });
    advance();
  }
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(2 * NL) : "memory");   // the first k tile has landed
  read_frags(KS(0), f0);
  MEFT_FENCE();

  int wg = wg0;
  for (;;) {
    const int my_tag = p.row_tag(tc, tc.m0 + wm + (lane & (TM / 2 - 1)));
    const int nk = tc.nk;
    k_tile(std::true_type{});
    for (int kt = 1; kt < nk; ++kt) k_tile(std::false_type{});

    // ---- epilogue out of the registers: see gemm_mfma.h -----------------------------------------------------------
    const bool odd = (lane & 1) != 0;
    // Every store is issued, to nowhere where nothing is to be stored: their number has to be known (see k_tile).
    const int ncol = tc.n0 + wn + (fr & ~1);
    const int lane_row = fc * 4 + (lane & 1);
    static_assert(P::kRowsLinear, "");
    const uint32_t ld = (uint32_t)p.out_ld(tc), es = P::kOutBf16 ? 2u : 4u;
    const uint32_t lane_at = (uint32_t)(p.row_off(tc, 1, tc.m0 + wm + lane_row) + ncol) * es;   // outputs are below 4 GB
    const unsigned long long ok_mask = __ballot(my_tag != 0);
    const int nj = p.out_cols(tc) - ncol;   // column pair 32 j is stored where 32 j < nj
#pragma unroll
    for (int i = 0; i < MI; ++i) {
#pragma unroll
      for (int qh = 0; qh < 2; ++qh) {
        uint32_t aux[4][NJ];
#pragma unroll
        for (int qq = 0; qq < 4; ++qq) {
          const int r = 2 * (qh * 4 + qq), rl = i * 32 + (r >> 2) * 8 + (r & 3) + lane_row;
#pragma unroll
          for (int j = 0; j < NJ; ++j) {
            if constexpr (P::kAux) aux[qq][j] = p.load_aux(tc, tc.m0 + wm + rl, ncol + 32 * j);
            else aux[qq][j] = 0u;
          }
        }
#pragma unroll
        for (int qq = 0; qq < 4; ++qq) {
          const int r = 2 * (qh * 4 + qq), rc = i * 32 + (r >> 2) * 8 + (r & 3);
          const bool ok = ((ok_mask >> (rc + lane_row)) & 1ull) != 0;
#pragma unroll
          for (int j = 0; j < NJ; ++j) {
            const uint32_t at = ok && 32 * j < nj ? lane_at + (uint32_t)(rc * ld + 32 * j) * es : kNowhere;
            if constexpr (P::kOutBf16) {
              // both rows' values of this lane's column are packed, one neighbour swap and one byte permute give
              // (column c | column c + 1 << 16) of the lane's row
              const uint32_t own = pack_bf16x2(acc[i][j][r], acc[i][j][r + 1]);
              const uint32_t nb = (uint32_t)__builtin_amdgcn_update_dpp((int)own, (int)own, 0xB1, 0xF, 0xF, true);
              const uint32_t pk = __builtin_amdgcn_perm(nb, own, odd ? 0x03020706u : 0x05040100u);
              __builtin_amdgcn_raw_buffer_store_b32(p.keep(pk, ncol + 32 * j, aux[qq][j]), rsrc_o, (int)at, 0, 0);
            } else {
              const float a = acc[i][j][r], b = acc[i][j][r + 1];
              const float an = __builtin_amdgcn_update_dpp(a, a, 0xB1, 0xF, 0xF, true);
              const float bn = __builtin_amdgcn_update_dpp(b, b, 0xB1, 0xF, 0xF, true);
              const u32x2 v = {__float_as_uint(odd ? bn : a), __float_as_uint(odd ? b : an)};
              __builtin_amdgcn_raw_buffer_store_b64(v, rsrc_o, (int)at, 0, 0);
            }
          }
        }
      }
    }
    since = 0;
    wg += step;
    if (!next_tile(fc_, wg, tc)) break;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // requests beyond the stream still write (zeros) to LDS
#undef KS
#undef MEFT_FENCE
}

}  // namespace meft
