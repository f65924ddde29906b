// Pieces shared by the kernels that multiply integers as signed 8-bit digits on
// v_mfma_i32_16x16x64_i8: register types, windows of a reversed digit string, and
// the recombination's multiply-add.
#pragma once
#include "device_common.h"

namespace pencil {

typedef int mx_v4i __attribute__((ext_vector_type(4)));
typedef uint32_t mx_u2 __attribute__((ext_vector_type(2)));
typedef uint32_t mx_u4 __attribute__((ext_vector_type(4)));

// Window o of the reversed bytes (r0 = bytes 0..3, r1 = bytes 4..7).
template <int O>
__device__ __forceinline__ uint32_t mx_window(uint32_t r0, uint32_t r1) {
  if constexpr (O < 0) return r0 << (-8 * O);
  else if constexpr (O == 0) return r0;
  else if constexpr (O < 4) return __builtin_amdgcn_alignbyte(r1, r0, O);
  else return r1 >> (8 * (O - 4));
}

// acc + d m for a 32-bit signed d, one v_mad_i64_i32 (m is kept opaque so that a
// power of two does not become a sign extension, a shift and an addition).
__device__ __forceinline__ int64_t mx_mad(int32_t d, int32_t m, int64_t acc) { return acc + (int64_t)d * m; }

}  // namespace pencil
