// sdtw_common.hpp -- device-side building blocks shared by the sDTW kernels.
//
// The DP cell (paper: Section 2, Eq. (1)):
//     D(i,j) = min{D(i-1,j), D(i,j-1), D(i-1,j-1)} + c(q_i, r_j)
// evaluated in binary32 as t = q - r; c = t*t (or |t|); D = min3 + c, every
// operation rounded to nearest-even (the library is built with
// -ffp-contract=off so no fused multiply-add is formed).  Each cell is a
// deterministic function of its three inputs, so any schedule of the cells
// yields identical bits.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sdtw {

constexpr int kWave = 64;            // CDNA wavefront width
constexpr int kRowCkpt = 256;        // row checkpoints: D(256k, 1..M) for 256k < N
constexpr int kSquared = 0;
constexpr int kAbsolute = 1;
// Squared difference with early pruning (the paper's Section 8 proposal):
// after the subtraction, a pair farther apart than the threshold tau is
// treated as unable to lie on the path and costs +inf, with no
// multiplication; otherwise the cost is t*t.
constexpr int kPruned = 2;

__device__ __forceinline__ float inf_f32() { return __builtin_huge_valf(); }

// Local cost c(q, r) for the cost kind (tau: the pruning threshold, used by
// kPruned only).
template <int KIND>
__device__ __forceinline__ float local_cost(float q, float r, float tau = 0.0f) {
  float t = q - r;
  if constexpr (KIND == kSquared) {
    return t * t;
  } else if constexpr (KIND == kPruned) {
    // Without a compare: (|t| - tau) * inf is +inf when |t| > tau, -inf when
    // |t| < tau and NaN when they are equal (the difference of two binary32
    // values is zero only when they are equal, subnormals being kept), and
    // the IEEE maximum ignores a NaN operand.  Every instruction reads only
    // vector registers, so all of them can dual-issue; a compare and select
    // would go through VCC, which cannot.
    const float w = (__builtin_fabsf(t) - tau) * inf_f32();
    return __builtin_fmaxf(t * t, w);
  } else {
    return __builtin_fabsf(t);
  }
}

// A wave-uniform value moved into a vector register.  The compiler would
// keep it in a scalar register, and VALU instructions that read a scalar
// register are not dual-issued on gfx950.
__device__ __forceinline__ float vgpr_copy(float x) {
  float v;
  asm("v_mov_b32 %0, %1" : "=v"(v) : "s"(x));
  return v;
}

// An empty asm statement that "modifies" a loaded value: the wait for the
// load is placed here, and no later use of the value can need one.
template <typename X>
__device__ __forceinline__ void in_register(X& x) {
  if constexpr (sizeof(X) == 4) {
    uint32_t w = __builtin_bit_cast(uint32_t, x);
    asm volatile("" : "+v"(w));
    x = __builtin_bit_cast(X, w);
  } else {
    uint32_t w = x;
    asm volatile("" : "+v"(w));
    x = (X)w;
  }
}

// One tile row of T lane values between registers and LDS, four at a time,
// in planes of four columns STRIDE words apart (4 for a row stored in one
// piece); every piece is 16-byte aligned.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <int STRIDE>
__device__ __forceinline__ int plane_at(int x, int t) {
  return (t >> 2) * STRIDE + 4 * x + (t & 3);
}

template <int T, int STRIDE, typename V>
__device__ __forceinline__ void tile_load(V (&dst)[T], const V* src) {
  static_assert(T % 4 == 0 && sizeof(V) == 4, "16-byte pieces");
#pragma unroll
  for (int t = 0; t < T; t += 4) {
    const u32x4 w = *reinterpret_cast<const u32x4*>(src + (t / 4) * STRIDE);
#pragma unroll
    for (int u = 0; u < 4; ++u) dst[t + u] = __builtin_bit_cast(V, (uint32_t)w[u]);
  }
}

template <int T, int STRIDE, typename V>
__device__ __forceinline__ void tile_store(V* dst, const V (&src)[T]) {
#pragma unroll
  for (int t = 0; t < T; t += 4) {
    u32x4 w;
#pragma unroll
    for (int u = 0; u < 4; ++u) w[u] = __builtin_bit_cast(uint32_t, src[t + u]);
    *reinterpret_cast<u32x4*>(dst + (t / 4) * STRIDE) = w;
  }
}

// Exact three-way minimum (one v_min3_f32).  Inputs are never NaN here: DP
// values start at 0 or +inf and every LDS slot a lane reads before its
// first tile is initialised (+inf boundaries, a zeroed reference ring).
__device__ __forceinline__ float min3(float a, float b, float c) {
  return __builtin_fminf(__builtin_fminf(a, b), c);
}

// Wavefront right shift by one lane (DPP wave_shr:1): lane l receives lane
// l-1's `v`; lane 0 keeps `lane0` (the row mask and bank mask enable every
// lane, and bound_ctrl is off so the invalid source lane leaves the old
// value in place).
__device__ __forceinline__ float wave_shr1(float lane0, float v) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, lane0),
                                         __builtin_bit_cast(int, v),
                                         0x138 /* wave_shr:1 */, 0xf, 0xf, false));
}

// Two such shifts: a takes va, b takes vb from the lane before (lane 0 keeps
// a and b).  On gfx950 two wavefronts of a SIMD issue a vector instruction
// each per quad-cycle as long as they stay in step; a DPP move cannot be
// paired, and moves that interleave with the other wavefront's arithmetic
// leave the two out of step for tens of instructions, so the pair goes out
// at raised priority.  (The two idle states in front are what a DPP read
// needs behind a vector write.)
template <typename V>
__device__ __forceinline__ void wave_shr1_pair(V& a, V va, V& b, V vb) {
  uint32_t x = __builtin_bit_cast(uint32_t, a), y = __builtin_bit_cast(uint32_t, b);
  asm volatile(
      "s_nop 1\n\t"
      "s_setprio 3\n\t"
      "v_mov_b32_dpp %0, %2 wave_shr:1 row_mask:0xf bank_mask:0xf\n\t"
      "v_mov_b32_dpp %1, %3 wave_shr:1 row_mask:0xf bank_mask:0xf\n\t"
      "s_setprio 0"
      : "+&v"(x), "+&v"(y)
      : "v"(__builtin_bit_cast(uint32_t, va)), "v"(__builtin_bit_cast(uint32_t, vb)));
  a = __builtin_bit_cast(V, x);
  b = __builtin_bit_cast(V, y);
}

template <int X>
constexpr int pow2_ceil() {
  int p = 1;
  while (p < X) p <<= 1;
  return p;
}

}  // namespace sdtw
