// Device-side helpers shared by the libmeft kernels (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace meft {

constexpr int kWave = 64;

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(4))) int32_t i32x4;
typedef u32x4 u32x4_dw __attribute__((aligned(4)));   // the same in memory where only four bytes are sure to be aligned

// ---- storage types -------------------------------------------------------------------------
struct bf16_t {
  uint16_t bits;
};

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t b) { return __uint_as_float(b << 16); }

// round to nearest, ties to even (inputs finite)
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return u >> 16;
}

// two floats -> two bf16 in one word (lo in bits 0..15), round to nearest even: one v_cvt_pk_bf16_f32 on gfx950
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_hw;
typedef __attribute__((ext_vector_type(2))) float f32x2_hw;
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  const f32x2_hw v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_hw));
}

// Eight consecutive elements of a row as floats.  Rows are 16-byte aligned and d % 8 == 0.
template <typename T>
struct Vec8;

template <>
struct Vec8<float> {
  static constexpr int kBytes = 32;
  static __device__ __forceinline__ void load(const float* p, float (&v)[8]) {
    const f32x4 a = *reinterpret_cast<const f32x4*>(p);
    const f32x4 b = *reinterpret_cast<const f32x4*>(p + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  }
  static __device__ __forceinline__ void store(float* p, const float (&v)[8]) {
    f32x4 a = {v[0], v[1], v[2], v[3]};
    f32x4 b = {v[4], v[5], v[6], v[7]};
    *reinterpret_cast<f32x4*>(p) = a;
    *reinterpret_cast<f32x4*>(p + 4) = b;
  }
};

template <>
struct Vec8<bf16_t> {
  static constexpr int kBytes = 16;
  static __device__ __forceinline__ void load(const bf16_t* p, float (&v)[8]) { widen(*reinterpret_cast<const u32x4*>(p), v); }
  // what nobody reads again
  static __device__ __forceinline__ void load_once(const bf16_t* p, float (&v)[8]) {
    widen(__builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p)), v);
  }
  static __device__ __forceinline__ void widen(u32x4 a, float (&v)[8]) {
    v[0] = __uint_as_float(a.x << 16); v[1] = __uint_as_float(a.x & 0xFFFF0000u);
    v[2] = __uint_as_float(a.y << 16); v[3] = __uint_as_float(a.y & 0xFFFF0000u);
    v[4] = __uint_as_float(a.z << 16); v[5] = __uint_as_float(a.z & 0xFFFF0000u);
    v[6] = __uint_as_float(a.w << 16); v[7] = __uint_as_float(a.w & 0xFFFF0000u);
  }
  static __device__ __forceinline__ void store(bf16_t* p, const float (&v)[8]) {
    u32x4 a;
    a.x = pack_bf16x2(v[0], v[1]);
    a.y = pack_bf16x2(v[2], v[3]);
    a.z = pack_bf16x2(v[4], v[5]);
    a.w = pack_bf16x2(v[6], v[7]);
    *reinterpret_cast<u32x4*>(p) = a;
  }
};

// One 16-byte word of a row as floats.  `store` is for finished rows, past L2, which keeps the slices of h and dOut that the
// per-pair kernels gather from (us per step, plain / nontemporal: 2048 tokens, one block of 65536 x 4096 2865 / 2823; 700 tokens,
// one of 16384 x 2048 227 / 211); `store_f32` for sums that are read again.
template <typename T>
struct Vec16;

template <>
struct Vec16<float> {
  static constexpr int kElems = 4;
  static __device__ __forceinline__ void unpack(u32x4 a, float (&v)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = __uint_as_float(a[i]);
  }
  static __device__ __forceinline__ void store(float* p, const float (&v)[4]) {
    __builtin_nontemporal_store((f32x4{v[0], v[1], v[2], v[3]}), reinterpret_cast<f32x4*>(p));
  }
  static __device__ __forceinline__ void store_f32(float* p, const float (&v)[4]) {
    *reinterpret_cast<f32x4*>(p) = f32x4{v[0], v[1], v[2], v[3]};
  }
};

template <>
struct Vec16<bf16_t> {
  static constexpr int kElems = 8;
  static __device__ __forceinline__ void unpack(u32x4 a, float (&v)[8]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[2 * i] = __uint_as_float(a[i] << 16);
      v[2 * i + 1] = __uint_as_float(a[i] & 0xFFFF0000u);
    }
  }
  static __device__ __forceinline__ void store(bf16_t* p, const float (&v)[8]) {
    const u32x4 a = {pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7])};
    __builtin_nontemporal_store(a, reinterpret_cast<u32x4*>(p));
  }
  static __device__ __forceinline__ void store_f32(float* p, const float (&v)[8]) { Vec8<float>::store(p, v); }
};

// ---- wave-level reductions -----------------------------------------------------------------
// sum over the wave, in every lane: DPP moves inside the rows of 16 lanes, then two lane permutes
__device__ __forceinline__ float wave_sum(float v) {
#define MEFT_DPP_ADDF(ctrl) v += __builtin_amdgcn_update_dpp(0.f, v, ctrl, 0xF, 0xF, false)
  MEFT_DPP_ADDF(0xB1);    // quad_perm [1,0,3,2]
  MEFT_DPP_ADDF(0x4E);    // quad_perm [2,3,0,1]
  MEFT_DPP_ADDF(0x141);   // row_half_mirror
  MEFT_DPP_ADDF(0x140);   // row_mirror
#undef MEFT_DPP_ADDF
  v += __shfl_xor(v, 16, kWave);
  return v + __shfl_xor(v, 32, kWave);
}

// eight sums at once: lane l receives the sum over the wave of v[l % 8].  Lanes hand the values they do not keep to a
// neighbour (23 vector instructions and two permutes instead of eight times four and two).
__device__ __forceinline__ float wave_sum8(const float (&v)[8]) {
  const int lane = threadIdx.x & 63;
  const bool b0 = (lane & 1) != 0, b1 = (lane & 2) != 0, b2 = (lane & 4) != 0;
  float a[4], c[2];
#define MEFT_DPP_GET(x, ctrl) __builtin_amdgcn_update_dpp(0.f, (x), ctrl, 0xF, 0xF, false)
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float give = b0 ? v[2 * i] : v[2 * i + 1];
    a[i] = (b0 ? v[2 * i + 1] : v[2 * i]) + MEFT_DPP_GET(give, 0xB1);   // quad_perm [1,0,3,2]
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const float give = b1 ? a[2 * i] : a[2 * i + 1];
    c[i] = (b1 ? a[2 * i + 1] : a[2 * i]) + MEFT_DPP_GET(give, 0x4E);   // quad_perm [2,3,0,1]
  }
  const float give = b2 ? c[0] : c[1];
  float r = (b2 ? c[1] : c[0]) + MEFT_DPP_GET(give, 0x124);             // row_ror:4, the quad four lanes away
  r += MEFT_DPP_GET(r, 0x128);                                           // row_ror:8
#undef MEFT_DPP_GET
  r += __shfl_xor(r, 16, kWave);
  return r + __shfl_xor(r, 32, kWave);
}

// orders a wave's own LDS accesses (writes by some lanes, then reads by others) without a workgroup barrier
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ unsigned long long wave_max_u64(unsigned long long v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const unsigned long long w = __shfl_xor(v, o, kWave);
    v = w > v ? w : v;
  }
  return v;
}

// inclusive prefix sum across the wave: DPP moves (row shifts, then the rows' totals broadcast), which stay in the vector
// unit; through LDS permutes a scan takes about 700 cycles, most of a selection pass or of a dispatch table
__device__ __forceinline__ int wave_incl_scan(int v) {
#define MEFT_DPP_ADD(ctrl, rows) v += __builtin_amdgcn_update_dpp(0, v, ctrl, rows, 0xF, false)
  MEFT_DPP_ADD(0x111, 0xF);   // row_shr:1
  MEFT_DPP_ADD(0x112, 0xF);   // row_shr:2
  MEFT_DPP_ADD(0x114, 0xF);   // row_shr:4
  MEFT_DPP_ADD(0x118, 0xF);   // row_shr:8
  MEFT_DPP_ADD(0x142, 0xA);   // row_bcast:15 into rows 1 and 3
  MEFT_DPP_ADD(0x143, 0xC);   // row_bcast:31 into rows 2 and 3
#undef MEFT_DPP_ADD
  return v;
}

// Monotone map float -> uint32: a > b  <=>  key(a) > key(b); -0 and +0 share a key.
__device__ __forceinline__ uint32_t order_key(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u << 1) == 0u) u = 0u;  // -0 -> +0
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float key_to_float(uint32_t k) {
  const uint32_t u = (k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k;
  return __uint_as_float(u);
}

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

}  // namespace meft
