// Wavefront-level helpers shared by the kernels: sums over the 64 lanes through DPP row
// butterflies, the ordered key of the LM-head argmax, and the bfloat16 rounding of stored values.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hh {

// 16 bytes of a matrix that one workgroup of a launch reads, once: a streaming load, so that the weights of a pass (0.9 GB
// and more) do not push out of the caches what the next small launches start with - activations, launch arguments, code.
// Decode passes of one sequence, two rounds: 0.5B shape, k = 2, 7.18 -> 6.69 ms; 3B shape, k = 4, 10.08 -> 9.59 ms.  Models
// that would fit the 256 MB cache gain as well (one sequence, 1 to 12 blocks of the 0.5B shape, k = 2: 2.5 to 7 %; one and two
// blocks of the 3B shape, k = 4: 2 and 6 %; four sequences: -1 to 1 %), so the rule looks at the type alone.  It loses where
// drafts of less than the cache alternate with a verification that loads plainly (two blocks of the 3B shape, the second one
// left out of the draft, k = 8: 2910 against 2838 us with one sequence, 3631 against 3567 with four).  Not for float32
// weights: models of that size stay in the cache from pass to pass (2 % slower).
__device__ __forceinline__ uint4 load_once16(const void* p) {
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  const u32x4 v = __builtin_nontemporal_load(static_cast<const u32x4*>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}

// Sum of four squares in one order wherever it stands (y's square is rounded, the others are added by fused operations).  As a plain expression the compiler picks per use which product it
// fuses, and rows that a kernel unrolls over were summed in different orders: equal rows of a batch with unequal bits.
__device__ __forceinline__ float sum_squares4(const float4& v) { return fmaf(v.w, v.w, fmaf(v.z, v.z, fmaf(v.x, v.x, v.y * v.y))); }

// v of lane l combined with the lane that a DPP control selects (row_shr, quad_perm, row_bcast ...)
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
// sum over each row of 16 lanes, left in every lane of the row
__device__ __forceinline__ float row16_sum(float v) {
  v += dpp_move<0xB1>(v);    // quad_perm [1,0,3,2]
  v += dpp_move<0x4E>(v);    // quad_perm [2,3,0,1]
  v += dpp_move<0x141>(v);   // row_half_mirror
  v += dpp_move<0x140>(v);   // row_mirror
  return v;
}
// largest of each 8 / 16 lanes' values, none of them negative, left in every one of them (as unsigned words: one instruction per step where
// the float maximum takes five, for moving and quieting its operands)
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_max(uint32_t u) { return max(u, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)u, CTRL, 0xf, 0xf, false)); }
__device__ __forceinline__ float lanes8_max(float v) { return __uint_as_float(dpp_max<0x141>(dpp_max<0x4E>(dpp_max<0xB1>(__float_as_uint(v))))); }
__device__ __forceinline__ float row16_max(float v) { return __uint_as_float(dpp_max<0x140>(__float_as_uint(lanes8_max(v)))); }
// sum over the 64 lanes (the four row totals added in row order), uniform result
__device__ __forceinline__ float wave_sum64(float v) {
  v = row16_sum(v);
  const int iv = __float_as_int(v);
  return (__int_as_float(__builtin_amdgcn_readlane(iv, 0)) + __int_as_float(__builtin_amdgcn_readlane(iv, 16))) +
         (__int_as_float(__builtin_amdgcn_readlane(iv, 32)) + __int_as_float(__builtin_amdgcn_readlane(iv, 48)));
}

// Key whose unsigned order is (larger value first, then lower index): the maximum over keys is the
// argmax with the lowest index among equal values.
__device__ __forceinline__ unsigned long long argmax_key(float v, int n) {
  uint32_t u = __float_as_uint(v);
  u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  return (static_cast<unsigned long long>(u) << 32) | static_cast<unsigned long long>(0xFFFFFFFFu - (uint32_t)n);
}

// float32 -> bfloat16 bits, round to nearest even (the rounding of every value stored as bf16)
__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf16_bits_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// v / d for d >= 1 (infinity counts as the largest finite value; above 2^126 the result is zero): the hardware's reciprocal and the
// quotient corrected by its remainder, 5 instructions where the IEEE division takes 10, and the same bits on the 2^20 values each of
// |v| < 0.5, 2, 8, 30 and 80 that were compared.  (The reciprocal corrected before it is multiplied, which rounds twice: rms error of the SiLU 5.0e-8 instead of
// 4.3e-8 for |v| < 0.5, a quarter of the bits others.)
__device__ __forceinline__ float div_above_one(float v, float d) {
  constexpr float kMax = 3.402823466e+38f;
  d = fminf(d, kMax);
  const float r = __builtin_amdgcn_rcpf(d), q = v * r;
  return fmaf(fminf(fmaf(-d, q, v), kMax), r, q);   // (the remainder of an infinite v is NaN)
}
// v * sigmoid(v) with the hardware exponential (within 1 ulp; the argument scaling adds |v| * 2^-24 relative): for every conv channel
// of every position.  Decode rounds 0.3 to 0.9 % faster than with the IEEE division, a walk of the matmul-form scan 4 %.
__device__ __forceinline__ float fast_silu(float v) { return div_above_one(v, 1.0f + __expf(-v)); }

}  // namespace hh
