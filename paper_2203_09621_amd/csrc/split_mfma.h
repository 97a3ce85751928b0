// The split forms' 16-bit operand types: the MFMA of one 16-wide k step and the
// factor 2^t that the hi part of A takes in registers.
#pragma once

#include "dmpt_internal.h"

namespace dmpt {

template <typename T16> struct Split16;

template <> struct Split16<_Float16> {
  typedef f16x8 V;
  static constexpr int kShift = kLoShiftF16;
  static __device__ __forceinline__ f32x16 mma(V a, V b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ V up(V a) {
    return a * (_Float16)(float)(1 << kShift);
  }
};

template <> struct Split16<__bf16> {
  typedef bf16x8 V;
  static constexpr int kShift = kLoShiftBF16;
  static __device__ __forceinline__ f32x16 mma(V a, V b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ V up(V a) { return a; }  // t = 0
};

}  // namespace dmpt
