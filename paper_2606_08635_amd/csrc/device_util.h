// Device-side helpers for gfx950 (CDNA4, 64-lane wavefronts).
#pragma once

#include <stdint.h>

#include <hip/hip_runtime.h>

namespace skv {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

enum : int { kFP16 = 0, kINT8 = 1, kINT4 = 2, kDROP = 3 };

// Row width in units of d/2 bytes and "is quantized" flag of each tier (0 for
// the code past kDROP that marks an absent token).
__device__ __forceinline__ uint32_t tier_units(int tr) { return (0x124u >> (4 * tr)) & 0xFu; }
__device__ __forceinline__ uint32_t tier_quant(int tr) { return (0x6u >> tr) & 1u; }

// Streaming (non-temporal) 16/8/4-byte global accesses.
__device__ __forceinline__ u32x4 ld_nt16(const void* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
}
__device__ __forceinline__ u32x2 ld_nt8(const void* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(p));
}
__device__ __forceinline__ uint32_t ld_nt4(const void* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const uint32_t*>(p));
}
__device__ __forceinline__ void st_nt16(void* p, u32x4 v) {
  __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(p));
}
__device__ __forceinline__ void st_nt8(void* p, u32x2 v) {
  __builtin_nontemporal_store(v, reinterpret_cast<u32x2*>(p));
}
__device__ __forceinline__ void st_nt4(void* p, uint32_t v) {
  __builtin_nontemporal_store(v, reinterpret_cast<uint32_t*>(p));
}

// DPP lane move inside 16-lane rows (row_mask/bank_mask all set).
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_mov(uint32_t v) {
  return static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(v), CTRL, 0xF, 0xF, true));
}

// The values of lanes i and i ^ 16 (lane_pair16) or i and i ^ 32
// (lane_pair32), the lower lane's as lo, in both lanes: gfx950's
// v_permlane16_swap / v_permlane32_swap, one vector instruction each instead
// of a shuffle through the LDS unit and its address arithmetic.  The lanes
// exchanged stay inside aligned groups of 32 (lane_pair16) or the wave
// (lane_pair32), and every lane of such a group in use must be active.
struct LanePair {
  uint32_t lo, hi;
};
__device__ __forceinline__ LanePair lane_pair16(uint32_t v) {
  const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  return LanePair{r[0], r[1]};
}
__device__ __forceinline__ LanePair lane_pair32(uint32_t v) {
  const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return LanePair{r[0], r[1]};
}

// Maximum over aligned groups of G consecutive lanes (G = 4, 8, 16 or 32);
// every lane of a group receives the group's maximum.  Must be called with
// every lane of each group active.
template <int G>
__device__ __forceinline__ uint32_t group_max(uint32_t v) {
  static_assert(G == 4 || G == 8 || G == 16 || G == 32, "group size");
  if constexpr (G == 32) {
    const LanePair p = lane_pair16(v);  // lanes i and i ^ 16
    v = max(p.lo, p.hi);
  }
  if constexpr (G >= 16) v = max(v, dpp_mov<0x140>(v));  // row_mirror: lane i <-> 15-i
  if constexpr (G >= 8) v = max(v, dpp_mov<0x141>(v));   // row_half_mirror: i <-> 7-i
  v = max(v, dpp_mov<0xB1>(v));                          // quad_perm [1,0,3,2]
  v = max(v, dpp_mov<0x4E>(v));                          // quad_perm [2,3,0,1]
  return v;
}

// Maximum over the wave's 64 lanes (all active), in every lane.
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
  const LanePair p = lane_pair32(group_max<32>(v));
  return max(p.lo, p.hi);
}

// Largest |x| of 8 binary16 values as a magnitude bit pattern (bits & 0x7FFF).
// For finite values the order of magnitude patterns is the order of |x|; any
// pattern >= 0x7C00 means an infinity or NaN is present.
__device__ __forceinline__ uint32_t absmax_bits8(u32x4 x) {
  const u16x2 m0 = __builtin_bit_cast(u16x2, x.x & 0x7FFF7FFFu);
  const u16x2 m1 = __builtin_bit_cast(u16x2, x.y & 0x7FFF7FFFu);
  const u16x2 m2 = __builtin_bit_cast(u16x2, x.z & 0x7FFF7FFFu);
  const u16x2 m3 = __builtin_bit_cast(u16x2, x.w & 0x7FFF7FFFu);
  const u16x2 m = __builtin_elementwise_max(__builtin_elementwise_max(m0, m1),
                                            __builtin_elementwise_max(m2, m3));
  return max(static_cast<uint32_t>(m.x), static_cast<uint32_t>(m.y));
}

__device__ __forceinline__ float half_lo(uint32_t w) {
  return static_cast<float>(__builtin_bit_cast(_Float16, static_cast<uint16_t>(w & 0xFFFFu)));
}
__device__ __forceinline__ float half_hi(uint32_t w) {
  return static_cast<float>(__builtin_bit_cast(_Float16, static_cast<uint16_t>(w >> 16)));
}
// RN32(h * r) and RN32(h - c) of the low (HI = 0) or high (HI = 1) binary16
// half of w: one mixed-precision FMA instead of a conversion and an operation
// (the same value, as the conversion is exact; a zero product is +0).
template <int HI>
__device__ __forceinline__ float half_mul(uint32_t w, float r) {
  float o;
  if constexpr (HI) asm("v_fma_mix_f32 %0, %1, %2, 0 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(o) : "v"(w), "v"(r));
  else asm("v_fma_mix_f32 %0, %1, %2, 0 op_sel_hi:[1,0,0]" : "=v"(o) : "v"(w), "v"(r));
  return o;
}
template <int HI>
__device__ __forceinline__ float half_sub(uint32_t w, float c) {
  float o;
  if constexpr (HI) asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(o) : "v"(w), "v"(c));
  else asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel_hi:[1,0,0]" : "=v"(o) : "v"(w), "v"(c));
  return o;
}
// A half of w less the binary16 value in the low half of h, rounded to binary32.
template <int HI>
__device__ __forceinline__ float half_diff(uint32_t w, uint32_t h) {
  float o;
  if constexpr (HI) asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[1,0,0] op_sel_hi:[1,0,1]" : "=v"(o) : "v"(w), "v"(h));
  else asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel_hi:[1,0,1]" : "=v"(o) : "v"(w), "v"(h));
  return o;
}
// max(|a|, |b|, m) of finite values.
__device__ __forceinline__ float max_magnitude(float a, float b, float m) {
  float o;
  asm("v_max3_f32 %0, |%1|, |%2|, %3" : "=v"(o) : "v"(a), "v"(b), "v"(m));
  return o;
}
__device__ __forceinline__ uint32_t half_bits(float f) {
  return __builtin_bit_cast(uint16_t, static_cast<_Float16>(f));
}
// Two binary32 values rounded (nearest-even) to binary16 and packed low|high.
__device__ __forceinline__ uint32_t pack_half2(float lo, float hi) {
  const uint16_t a = __builtin_bit_cast(uint16_t, static_cast<_Float16>(lo));
  const uint16_t b = __builtin_bit_cast(uint16_t, static_cast<_Float16>(hi));
  return static_cast<uint32_t>(a) | (static_cast<uint32_t>(b) << 16);
}

// Inclusive prefix sum over the wave's 64 lanes (all active) by DPP lane moves:
// shifts inside the 16-lane rows, then the last lane of row 0 and 2 broadcast
// to the next row and that of row 1 to rows 2 and 3.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_shift(uint32_t v) {
  return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, ROWS, 0xF, false));
}
__device__ __forceinline__ uint32_t row_inclusive_scan(uint32_t x) {  // the 16 lanes of a row
  x += dpp_shift<0x111, 0xF>(x);  // row_shr:1
  x += dpp_shift<0x112, 0xF>(x);  // row_shr:2
  x += dpp_shift<0x114, 0xF>(x);  // row_shr:4
  x += dpp_shift<0x118, 0xF>(x);  // row_shr:8
  return x;
}
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t x) {
  x = row_inclusive_scan(x);
  x += dpp_shift<0x142, 0xA>(x);  // row_bcast:15
  x += dpp_shift<0x143, 0xC>(x);  // row_bcast:31
  return x;
}

// Exclusive prefix sum of one 32-bit value per thread over a block's first 256
// threads (4 wavefronts).  `scratch` holds at least 4 words of shared memory,
// not written again before the caller's next barrier.  Contains one
// __syncthreads(); every thread of the block must call it.
__device__ __forceinline__ uint32_t block_exclusive_scan_256(uint32_t x, uint32_t* scratch) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t inc = wave_inclusive_scan(x);
  if (lane == 63 && wave < 4) scratch[wave] = inc;
  __syncthreads();
  uint32_t base = 0;
#pragma unroll
  for (int w = 0; w < 3; ++w) base += (w < wave) ? scratch[w] : 0u;
  return base + inc - x;
}

}  // namespace skv
