// Exchanges between the lanes of a wavefront with DPP: what the windowed kernels use to settle a
// request that is spread over several lanes, and to add up what a wavefront admits.
#pragma once

#include "sweep_kernels.hpp"

namespace maaso {

__device__ __forceinline__ float lane_value(float v, int l) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}

// `old` with lane l (uniform) holding v (uniform): v_writelane.  Where the compiler has no builtin for it, the
// intrinsic by its name, which carries the type since LLVM 19; with any other compiler a compare and a select.
#if __has_builtin(__builtin_amdgcn_writelane)
__device__ __forceinline__ int with_lane(int old, int l, int v) { return __builtin_amdgcn_writelane(v, l, old); }
#elif __clang_major__ >= 19
__device__ int maaso_writelane(int v, int l, int old) __asm("llvm.amdgcn.writelane.i32");
__device__ __forceinline__ int with_lane(int old, int l, int v) { return maaso_writelane(v, l, old); }
#else
__device__ __forceinline__ int with_lane(int old, int l, int v) { return (int)__lane_id() == l ? v : old; }
#endif
__device__ __forceinline__ int with_lane(int old, int l, float v) { return with_lane(old, l, __builtin_bit_cast(int, v)); }

// At the head of a branch that is hardly ever taken: keeps the compiler from working out both sides of
// it and selecting.
__device__ __forceinline__ void rare_path() { asm volatile(""); }

// A non-negative time in ticks of 2^-20 s, rounded to nearest; `narrow`: known to be below 2^32 ticks.
__device__ __forceinline__ unsigned long long to_ticks(float seconds, bool narrow) {
  const float x = seconds * 1048576.0f;
  unsigned long long t = (unsigned long long)(uint32_t)rintf(x);
  if (!narrow) {
    rare_path();
    t = (unsigned long long)__float2ll_rn(x);
  }
  return t;
}

// x = OP(x, x of the lane that the DPP control CTRL names), one instruction.  A DPP operand written by
// the vector instruction just before needs two wait states, which the assembler does not add inside
// an asm statement: hence the s_nop.
// ROWS: mask of the 16-lane rows that are written; the others keep their value.
#define MAASO_DPP_FOLD_ROWS(OP, X, CTRL, ROWS) \
  asm("s_nop 1\n\t" OP " %0, %0, %0 " CTRL " row_mask:" ROWS " bank_mask:0xf" : "+v"(X))
#define MAASO_DPP_FOLD(OP, X, CTRL) MAASO_DPP_FOLD_ROWS(OP, X, CTRL, "0xf")

// Maximum (v_max_f32: a NaN operand loses) / unsigned minimum over groups of LPR consecutive lanes
// (a power of two up to 64); every lane ends with the group's value.  Up to 16 lanes the partner
// lanes are reached with DPP controls - lane ^ 1, lane ^ 2, then the mirrored quad of the 8 and the
// mirrored half of the 16-lane row - beyond that through LDS permutes.
template <int LPR>
__device__ __forceinline__ float max_lanes(float m) {
  if (LPR >= 2) MAASO_DPP_FOLD("v_max_f32_dpp", m, "quad_perm:[1,0,3,2]");
  if (LPR >= 4) MAASO_DPP_FOLD("v_max_f32_dpp", m, "quad_perm:[2,3,0,1]");
  if (LPR >= 8) MAASO_DPP_FOLD("v_max_f32_dpp", m, "row_half_mirror");
  if (LPR >= 16) MAASO_DPP_FOLD("v_max_f32_dpp", m, "row_mirror");
  if (LPR >= 32) m = max_no_nan(m, __shfl_xor(m, 16));
  if (LPR >= 64) m = max_no_nan(m, __shfl_xor(m, 32));
  return m;
}

template <int LPR>
__device__ __forceinline__ uint32_t min_lanes(uint32_t c) {
  if (LPR >= 2) MAASO_DPP_FOLD("v_min_u32_dpp", c, "quad_perm:[1,0,3,2]");
  if (LPR >= 4) MAASO_DPP_FOLD("v_min_u32_dpp", c, "quad_perm:[2,3,0,1]");
  if (LPR >= 8) MAASO_DPP_FOLD("v_min_u32_dpp", c, "row_half_mirror");
  if (LPR >= 16) MAASO_DPP_FOLD("v_min_u32_dpp", c, "row_mirror");
  if (LPR >= 32) c = min(c, (uint32_t)__shfl_xor((int)c, 16));
  if (LPR >= 64) c = min(c, (uint32_t)__shfl_xor((int)c, 32));
  return c;
}

// Arg-max of (slack, index) over groups of LPR consecutive lanes, lowest index among equal slacks;
// every lane ends with the winner.  Two reductions of one instruction per step: the largest slack,
// then the lowest index among the lanes that hold it.  A lane that has seen no slack above -inf
// carries index -1; when the maximum is -inf every lane of the group does, and -1 (the largest
// unsigned value) is what comes out.
template <int LPR>
__device__ __forceinline__ void argmax_lanes(float& s, int32_t& i) {
  const float m = max_lanes<LPR>(s);
  const uint32_t c = (s == m) ? (uint32_t)i : 0xffffffffu;
  i = (int32_t)min_lanes<LPR>(c);
  s = m;
}

// Sum of a 32-bit value over the wavefront (the caller makes sure it cannot overflow), as a uniform
// value: four DPP steps give every lane its row's sum, two row broadcasts carry the rows' sums into
// lane 63.  Six dependent vector additions instead of six trips through the LDS permute network.
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v) {
  MAASO_DPP_FOLD("v_add_u32_dpp", v, "quad_perm:[1,0,3,2]");
  MAASO_DPP_FOLD("v_add_u32_dpp", v, "quad_perm:[2,3,0,1]");
  MAASO_DPP_FOLD("v_add_u32_dpp", v, "row_half_mirror");
  MAASO_DPP_FOLD("v_add_u32_dpp", v, "row_mirror");
  MAASO_DPP_FOLD_ROWS("v_add_u32_dpp", v, "row_bcast:15", "0xa");
  MAASO_DPP_FOLD_ROWS("v_add_u32_dpp", v, "row_bcast:31", "0xc");
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// The sums of two values, each as wave_sum_u32: the steps of one fill the wait states of the other.
__device__ __forceinline__ void wave_sum_pair(uint32_t& x, uint32_t& y) {
  asm("s_nop 1\n\t"
      "v_add_u32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "v_add_u32_dpp %1, %1, %1 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 0\n\t"
      "v_add_u32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
      "v_add_u32_dpp %1, %1, %1 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 0\n\t"
      "v_add_u32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
      "v_add_u32_dpp %1, %1, %1 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 0\n\t"
      "v_add_u32_dpp %0, %0, %0 row_mirror row_mask:0xf bank_mask:0xf\n\t"
      "v_add_u32_dpp %1, %1, %1 row_mirror row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 0\n\t"
      "v_add_u32_dpp %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0xf\n\t"
      "v_add_u32_dpp %1, %1, %1 row_bcast:15 row_mask:0xa bank_mask:0xf\n\t"
      "s_nop 0\n\t"
      "v_add_u32_dpp %0, %0, %0 row_bcast:31 row_mask:0xc bank_mask:0xf\n\t"
      "v_add_u32_dpp %1, %1, %1 row_bcast:31 row_mask:0xc bank_mask:0xf"
      : "+v"(x), "+v"(y));
  x = (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
  y = (uint32_t)__builtin_amdgcn_readlane((int)y, 63);
}

// Sum over the wavefront of per-lane tick counts, uniform: in 32 bits when no lane holds 2^26 ticks (64 s
// of prefill) or more, the usual case; else 26 bits at a time.
__device__ __forceinline__ unsigned long long wave_sum_ticks(unsigned long long t) {
  constexpr uint32_t kPart = (1u << 26) - 1u;
  unsigned long long sum = wave_sum_u32((uint32_t)t & kPart);
  if (lane_mask((t >> 26) != 0ull) != 0ull) {
    sum += (unsigned long long)wave_sum_u32((uint32_t)(t >> 26) & kPart) << 26;
    sum += (unsigned long long)wave_sum_u32((uint32_t)(t >> 52)) << 52;
  }
  return sum;
}

}  // namespace maaso
