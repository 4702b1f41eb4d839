// Float products on the bfloat16 matrix cores (fused.hip, edge_grad.hip,
// dense.hip): each operand is split into three bfloat16 parts, x = hi + mid + lo
// exactly (8 + 8 + 8 bits hold the 24; from about 2^-110 down the lowest fall under
// the smallest bfloat16), and of the nine cross products the six
// that reach 2^-24 of the product are summed in float.  An infinite operand
// splits into an infinity and NaN, so its products are NaN, as is a finite
// one's that rounds to infinity in bfloat16 (above 2^128 - 2^119).
#pragma once

#include <hip/hip_runtime.h>

namespace e2f {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef __bf16 v2b __attribute__((ext_vector_type(2)));
typedef __bf16 v8b __attribute__((ext_vector_type(8)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));

// Two floats as three words of bfloat16 pairs: hi and mid rounded to nearest, lo
// the rest.
__device__ __forceinline__ void split_pair(float x, float y, unsigned& hi, unsigned& mid, unsigned& lo) {
  hi = __builtin_bit_cast(unsigned, __builtin_convertvector((v2f){x, y}, v2b));
  const float rx = x - __uint_as_float(hi << 16), ry = y - __uint_as_float(hi & 0xffff0000u);
  mid = __builtin_bit_cast(unsigned, __builtin_convertvector((v2f){rx, ry}, v2b));
  const float sx = rx - __uint_as_float(mid << 16), sy = ry - __uint_as_float(mid & 0xffff0000u);
  lo = __builtin_bit_cast(unsigned, __builtin_convertvector((v2f){sx, sy}, v2b));
}

__device__ __forceinline__ v4f mfma_bf16(v4u a, v4u b, v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8b, a), __builtin_bit_cast(v8b, b), c, 0, 0, 0);
}

}  // namespace e2f
