// fp32 operands on the bf16 matrix cores: x = h + m + l exactly, each part the
// bf16 rounding of what the parts before it leave (8 + 8 + 8 significand bits
// hold fp32's 24).
#pragma once

#include "device_util.h"

namespace pinsage {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

struct Split3 {
  u32x4 p[3];
};

// Parts of the eight fp32 values u[0..3], v[0..3].
__device__ __forceinline__ Split3 split3(const u32x4& u, const u32x4& v) {
  Split3 s;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    float x0 = __uint_as_float(q < 2 ? u[2 * q] : v[2 * q - 4]);
    float x1 = __uint_as_float(q < 2 ? u[2 * q + 1] : v[2 * q - 3]);
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      const uint32_t w = pack_bf16x2(x0, x1);
      s.p[t][q] = w;
      if (t < 2) {
        x0 -= __uint_as_float(w << 16);
        x1 -= __uint_as_float(w & 0xFFFF0000u);
      }
    }
  }
  return s;
}

// The six products of parts that matter, smallest first: (2,0) (0,2) (1,1)
// (1,0) (0,1) (0,0); the three left out are below 2^-25 of the product.
__device__ constexpr int split_b(int t) { return t == 0 ? 2 : (t == 2 || t == 3 ? 1 : 0); }
__device__ constexpr int split_a(int t) { return t == 1 ? 2 : (t == 2 || t == 4 ? 1 : 0); }

}  // namespace pinsage
