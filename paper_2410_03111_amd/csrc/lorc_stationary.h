// Internal: what the two split kernels with the key factor in registers share (lorc_decode_stat.hip, lorc_decode_stat768.hip).
#ifndef LORC_STATIONARY_H_
#define LORC_STATIONARY_H_

#include "lorc_device.h"

namespace lorc {

constexpr float kNegInfS = -__builtin_huge_valf();
constexpr float kBelow = 24.0f;  // log2 of the largest weight that an earlier tile may have next to a later one's 1
constexpr double kInvTwoPi = 0.15915494309189533576888;

constexpr int kStatWaves = 8;          // two per SIMD
constexpr int kStatThreads = 64 * kStatWaves;
constexpr int kStatMaxHeads = 16;      // query heads per workgroup: 2 KV heads x G <= 8
constexpr int kStatMaxTiles = 512;     // pages one workgroup walks at most (their ids live in LDS)
constexpr int kStatQPitch = 68;        // (x, y) query pairs of 4 bytes per head row in LDS: 64, and 4 that shift the next row's banks

typedef __attribute__((ext_vector_type(4))) float f32x4s;
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;

// D[16x16] += A[16x32] B[32x16].  Lane l supplies A[m = l%16][k = 8*(l/16) .. +7] and B[k = 8*(l/16) .. +7][n = l%16];
// it receives D[m = 4*(l/16) + j][n = l%16] in register j.
__device__ __forceinline__ f32x4s mfma16(bf16x8 a, bf16x8 b, f32x4s c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Maximum over rows of 16 lanes, step by step (the lane exchanges of half_wave_peer), in one vector instruction per step: the
// exchange is the operand modifier of the maximum.  (The two wait states cover the exchange of a value just written.)
template <int STEP>
__device__ __forceinline__ float row_max_step(float v) {
  float r;
  if constexpr (STEP == 0) asm("s_nop 1\n\tv_max_f32_dpp %0, %1, %1 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf" : "=v"(r) : "v"(v));
  if constexpr (STEP == 1) asm("s_nop 1\n\tv_max_f32_dpp %0, %1, %1 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf" : "=v"(r) : "v"(v));
  if constexpr (STEP == 2) asm("s_nop 1\n\tv_max_f32_dpp %0, %1, %1 row_ror:4 row_mask:0xf bank_mask:0xf" : "=v"(r) : "v"(v));
  if constexpr (STEP == 3) asm("s_nop 1\n\tv_max_f32_dpp %0, %1, %1 row_ror:8 row_mask:0xf bank_mask:0xf" : "=v"(r) : "v"(v));
  return r;
}

}  // namespace lorc
#endif  // LORC_STATIONARY_H_
